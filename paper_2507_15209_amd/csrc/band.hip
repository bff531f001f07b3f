// band.hip -- grid summation with the connection coefficients (Eqs. con-coeff,
// SFC-3PCF), forward and adjoint, both bases.
//
// The summation sum_x p_x sum_{s,t} Gamma(s, t) a_b1(x + s) conj(a_b2(x + t)) is a
// trilinear form that factors over the axes.  Along y and z it is written as a
// sum over q points per cell, at which the fields and the primary are short
// filters of the grid values (BandRule: for the B-spline the 4-point rule that
// integrates every C^2 spline of degree 9 on unit cells exactly, for
// Daubechies-4 the five eigenvectors of the coefficient matrix).  Along x it
// keeps the band form: with the primary filtered onto a (y, z) point,
//   M_d(x) = sum_j gamma(-j, -j - d) p(x + j),
//   sum_x sum_d M_d(x) a_b1(x) conj(a_b2(x - d)) + (b1 <-> b2, d > 0),
// so that a point costs one product per x plane instead of one per x node and
// the march along x needs no halo.  Against points on all three axes this is a
// quarter of the contraction's products and half of the interpolation.
#include "fft_core.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

#include <hip/hip_runtime.h>

#include <type_traits>

namespace mp3 {

namespace {

// BandRule in the working precision (kernel argument)
template <typename T, int Q, int TP, int H>
struct RuleT {
  T f[Q][TP], p[Q][TP], g[H + 1][2 * H + 1];
};

template <typename T, int Q, int TP, int H>
RuleT<T, Q, TP, H> rule_of(const BandRule& r) {
  RuleT<T, Q, TP, H> o;
  for (int s = 0; s < Q; ++s)
    for (int t = 0; t < TP; ++t) {
      o.f[s][t] = (T)r.f[s][t];
      o.p[s][t] = (T)r.p[s][t];
    }
  for (int d = 0; d <= H; ++d)
    for (int j = 0; j <= 2 * H; ++j) o.g[d][j] = (T)r.g[d][j];
  return o;
}

__device__ __forceinline__ int wrap_n(int i, int n) { return i & (n - 1); }   // n is a power of two

template <typename T, int Q, int TP, int TY, int NH>
struct ContractLds {
  static constexpr int ZC = 4, ZG = ZC + TP - 1, YG = TY + TP - 1, W = TY * Q, NODES = ZC * Q;
  size_t C, P, V, Vp, M, total;
  __host__ __device__ ContractLds(int nl) {
    size_t o = 0;
    auto take = [&](size_t b) { size_t r = o; o = (o + b + 15) & ~(size_t)15; return r; };
    C = take((size_t)2 * YG * ZG * nl * sizeof(c2<T>));
    P = take((size_t)2 * YG * ZG * sizeof(T));
    V = take((size_t)W * ZG * 16 * NH * sizeof(c2<T>));
    Vp = take((size_t)W * 16 * sizeof(T));
    M = take((size_t)W * NODES * 4 * sizeof(T));
    const size_t red = (size_t)W * 256 * sizeof(double) + (size_t)NH * NH * 256 * sizeof(double);
    total = o > red ? o : red;
  }
};

// Forward contraction.  A workgroup marches along x over a tile of TY x 4 cells
// in (y, z); wave (cell row yc, y point sy) holds the points of four z cells:
// lane l is bin l % 16 (and 16 + l % 16 when NH = 2) of z cell l / 16, which is
// the operand layout of the 16x16x4 matrix instructions, so fields and banded
// fields go from registers to the matrix cores without an exchange.  Per plane:
// y filter (LDS plane -> the wave's rows), z filter (rows -> Q points in
// registers), the band over the last H planes held in registers, products.
// Only the half band d >= 0 is applied (d = 0 at half weight): the sum over
// the transposed pairs is T + T^T, taken once at the end.
// Bound by instruction issue (vector ALU, LDS and matrix products share a wave's
// issue slots); partial sums are float32, as the fields are, over a workgroup's marches
// (two at 256^3 with 4096 workgroups), float64 beyond.  float64 with 17..32 bins spills 100 to 113
// of its 256 registers (two bin halves of the window).  Against 5^3 Gauss points per cell interpolated into LDS rows: 256^3, 20
// bins 160.7 -> 17.8 ms per item; 128^3, 15 bins 14.0 -> 0.85 ms.
template <typename T, int Q, int TP, int H, int TY, int NH>
__global__ void __launch_bounds__(TY* Q * 64)
    k_band_contract(const c2<T>* fields, const T* prim, int n, int nbt, int a0, int na, int c0, int nl, int off,
                    RuleT<T, Q, TP, H> rule, int nseg, int pair, double* partials) {
  using L_ = ContractLds<T, Q, TP, TY, NH>;
  constexpr int ZC = L_::ZC, ZG = L_::ZG, YG = L_::YG, NODES = L_::NODES, NT = TY * Q * 64, W = TY * Q;
  constexpr int CELLS = YG * ZG, PF = (CELLS * 16 * NH + NT - 1) / NT, WIN = H + 1;
  using A4 = typename acc4<T>::type;
  extern __shared__ __align__(16) char smem[];
  const L_ L(nl);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int yc = wave / Q, sy = wave % Q;
  const int bl = lane & 15, kl = lane >> 4;
  c2<T>* V = reinterpret_cast<c2<T>*>(smem + L.V) + (size_t)wave * ZG * 16 * NH;
  T* Vp = reinterpret_cast<T*>(smem + L.Vp) + wave * 16;
  T* Ml = reinterpret_cast<T*>(smem + L.M) + (size_t)wave * NODES * 4;
  const long long n2 = (long long)n * n;
  const c2<T>* fm = fields + (long long)blockIdx.y * n2 * n * nbt;
  const T* pm = prim + (long long)blockIdx.y * n2 * n;
  // this wave's y filters; this lane's band entry: point j, shift dl
  T wy[TP], pwy[TP];
#pragma unroll
  for (int t = 0; t < TP; ++t) {
    wy[t] = rule.f[sy][t];
    pwy[t] = rule.p[sy][t];
  }
  const int dl = lane / NODES <= H ? lane / NODES : H;
  const int node = lane % NODES, nzc = node / Q, ns = node % Q;
  const bool has_m = lane / NODES <= H;
  T pz[TP], gl[2 * H + 1];
#pragma unroll
  for (int t = 0; t < TP; ++t) pz[t] = rule.p[ns][t];
#pragma unroll
  for (int j = 0; j <= 2 * H; ++j) gl[j] = rule.g[dl][j] * (dl == 0 ? (T)0.5 : (T)1);
  int bc[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) bc[h] = 16 * h + bl < nl ? 16 * h + bl : 0;   // absent bins: dropped at the end
  // the real and the imaginary parts' products apart: the parts of a pair item are two multipoles' fields
  A4 acc[2][NH][NH];
#pragma unroll
  for (int i = 0; i < NH; ++i)
#pragma unroll
    for (int k = 0; k < NH; ++k) acc[0][i][k] = acc[1][i][k] = A4{0, 0, 0, 0};

  const int tz = n / ZC, ty = n / TY, ntask = ty * tz * nseg, seg = n / nseg;
  for (int task0 = blockIdx.x; task0 < ntask; task0 += gridDim.x) {
    const int task = xcd_order(task0, ntask);
    const int sg = task % nseg, tile = task / nseg;
    const int y0 = (tile / tz) * TY + off, z0 = (tile % tz) * ZC + off, x0 = sg * seg;
    int src[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int e = tid + i * NT, bb = e % nl, cell = e / nl;
      const int yy = wrap_n(y0 + cell / ZG, n), zz = wrap_n(z0 + cell % ZG, n);
      src[i] = cell < CELLS ? (yy * n + zz) * nbt + (bb < na ? a0 + bb : c0 + bb - na) : -1;
    }
    int psrc = -1;
    if (tid < CELLS) psrc = wrap_n(y0 + tid / ZG, n) * n + wrap_n(z0 + tid % ZG, n);
    c2<T> win[NH][WIN][Q];
    T pr[2 * H + 1];
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int i = 0; i < WIN; ++i)
#pragma unroll
        for (int s = 0; s < Q; ++s) win[h][i][s] = mk<T>(0, 0);
#pragma unroll
    for (int j = 0; j <= 2 * H; ++j) pr[j] = 0;
    c2<T> nextc[PF];
    T nextp = 0;
    auto fetch = [&](int x) {   // fields of plane x, primary of plane x + H
      const c2<T>* fp = fm + (long long)wrap_n(x, n) * n2 * nbt;
#pragma unroll
      for (int i = 0; i < PF; ++i) nextc[i] = src[i] >= 0 ? fp[src[i]] : mk<T>(0, 0);
      if (psrc >= 0) nextp = pm[(long long)wrap_n(x + H, n) * n2 + psrc];
    };
    fetch(x0 - 2 * H);
    // planes x0 - 2 H .. x0 - H - 1 only fill the primary's window, the next H the fields'
    const int steps = 2 * H + seg;
    for (int st0 = 0; st0 < steps; st0 += WIN) {
#pragma unroll
      for (int u = 0; u < WIN; ++u) {
        const int st = st0 + u, x = x0 - 2 * H + st;
        if (st < steps) {
          // keep the lane's LDS addresses inside the step: hoisted out of the loop they would pin registers
          int b = bl, kq = kl;
          asm volatile("" : "+v"(b), "+v"(kq));
          c2<T>* C = reinterpret_cast<c2<T>*>(smem + L.C) + (size_t)(st & 1) * CELLS * nl;
          T* P = reinterpret_cast<T*>(smem + L.P) + (st & 1) * CELLS;
#pragma unroll
          for (int i = 0; i < PF; ++i)
            if (src[i] >= 0) C[tid + i * NT] = nextc[i];
          if (psrc >= 0) P[tid] = nextp;
          __syncthreads();
          if (st + 1 < steps) fetch(x + 1);
          // y filters
          if (st >= H) {
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
              for (int it = 0; it < (ZG + 3) / 4; ++it) {
                const int zg = kq + 4 * it;
                if (zg < ZG) {
                  c2<T> a = mk<T>(0, 0);
#pragma unroll
                  for (int t = 0; t < TP; ++t) {
                    const c2<T> v = C[((yc + t) * ZG + zg) * nl + bc[h]];
                    a.x += wy[t] * v.x;
                    a.y += wy[t] * v.y;
                  }
                  V[(zg * NH + h) * 16 + b] = a;
                }
              }
          }
          if (lane < ZG) {
            T a = 0;
#pragma unroll
            for (int t = 0; t < TP; ++t) a += pwy[t] * P[(yc + t) * ZG + lane];
            Vp[lane] = a;
          }
          col_sync<true>();
          // band coefficients of the wave's points at plane x
#pragma unroll
          for (int j = 0; j < 2 * H; ++j) pr[j] = pr[j + 1];
          {
            T a = 0;
#pragma unroll
            for (int t = 0; t < TP; ++t) a += pz[t] * Vp[nzc + t];
            pr[2 * H] = a;
          }
          if (st >= H) {
            T m = 0;
#pragma unroll
            for (int j = 0; j <= 2 * H; ++j) m += gl[j] * pr[j];
            if (has_m) Ml[node * 4 + dl] = m;
            col_sync<true>();
            // z filter: the wave's points in registers
#pragma unroll
            for (int h = 0; h < NH; ++h) {
              c2<T> v[TP];
#pragma unroll
              for (int t = 0; t < TP; ++t) v[t] = V[((kq + t) * NH + h) * 16 + b];
#pragma unroll
              for (int s = 0; s < Q; ++s) {
                c2<T> a = mk<T>(0, 0);
#pragma unroll
                for (int t = 0; t < TP; ++t) {
                  a.x += rule.f[s][t] * v[t].x;
                  a.y += rule.f[s][t] * v[t].y;
                }
                win[h][u][s] = a;
              }
            }
            if (st >= 2 * H) {
#pragma unroll
              for (int s = 0; s < Q; ++s) {
                __builtin_amdgcn_sched_barrier(0);   // one point's coefficients in registers at a time
                T md[4];
#pragma unroll
                for (int d = 0; d <= H; ++d) md[d] = Ml[(kq * Q + s) * 4 + d];
                c2<T> g[NH];
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                  g[h] = mk<T>(0, 0);
#pragma unroll
                  for (int d = 0; d <= H; ++d) {
                    const c2<T> w = win[h][(u + WIN - d) % WIN][s];
                    g[h].x += md[d] * w.x;
                    g[h].y += md[d] * w.y;
                  }
                }
                // the products of one part on every block before the other's: dependent issues stay apart
#pragma unroll
                for (int h1 = 0; h1 < NH; ++h1)
#pragma unroll
                  for (int h2 = 0; h2 < NH; ++h2) acc[0][h1][h2] = mfma16(win[h1][u][s].x, g[h2].x, acc[0][h1][h2]);
#pragma unroll
                for (int h1 = 0; h1 < NH; ++h1)
#pragma unroll
                  for (int h2 = 0; h2 < NH; ++h2) acc[1][h1][h2] = mfma16(win[h1][u][s].y, g[h2].y, acc[1][h1][h2]);
              }
            }
          }
        }
      }
    }
    __syncthreads();   // the next task refills both planes
  }
  // T[b1][b2] over the waves in float64, then T + T^T; a pair item's parts one after the other
  double* red = reinterpret_cast<double*>(smem);
  double* tt = red + W * 256;   // [NH][NH][16][16]
  const int parts = pair ? 2 : 1;
  for (int part = 0; part < parts; ++part) {
#pragma unroll
    for (int h1 = 0; h1 < NH; ++h1)
#pragma unroll
      for (int h2 = 0; h2 < NH; ++h2) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const double re = (double)acc[0][h1][h2][i], im = (double)acc[1][h1][h2][i];
          red[wave * 256 + mfma_row<T>(lane, i) * 16 + bl] = !pair ? re + im : part == 0 ? re : im;
        }
        __syncthreads();
        for (int e = tid; e < 256; e += NT) {
          double s = 0.0;
          for (int w = 0; w < W; ++w) s += red[w * 256 + e];
          tt[(h1 * NH + h2) * 256 + e] = s;
        }
      }
    __syncthreads();
    double* out = partials + (((long long)blockIdx.y * gridDim.x + blockIdx.x) * parts + part) * nl * nl;
    for (int e = tid; e < nl * nl; e += NT) {
      const int b1 = e / nl, b2 = e % nl;
      out[e] = tt[((b1 / 16) * NH + b2 / 16) * 256 + (b1 % 16) * 16 + b2 % 16] +
               tt[((b2 / 16) * NH + b1 / 16) * 256 + (b2 % 16) * 16 + b1 % 16];
    }
  }
}

// lane l of a row of 16: the value of lane l + K (left) or l - K (right) of the row, 0 beyond it
template <int K> __device__ __forceinline__ float row_left(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x100 + K, 0xf, 0xf, true));
}
template <int K> __device__ __forceinline__ float row_right(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x110 + K, 0xf, 0xf, true));
}
template <int K> __device__ __forceinline__ double row_left(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x100 + K, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x100 + K, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <int K> __device__ __forceinline__ double row_right(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x110 + K, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x110 + K, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// z neighbours of a row of 16 cells: taps v[t](z) = w(z + t), t < TP, from the row's own values a
// (w(z), z < 16) and the halo h (w(16 + z) in the first lanes)
template <int TP, int T0, typename T> __device__ __forceinline__ void row_taps(T a, T h, T* v) {
  if constexpr (T0 < TP) {
    if constexpr (T0 == 0) v[0] = a;
    else v[T0] = row_left<T0>(a) + row_right<16 - T0>(h);
    row_taps<TP, T0 + 1, T>(a, h, v);
  }
}
// the transpose: out(z) = sum_t o[t](z - t) for z < 16 into a, for 16 <= z into the first lanes of h
template <int TP, int T0, typename T> __device__ __forceinline__ void row_taps_t(const T* o, T& a, T& h) {
  if constexpr (T0 < TP) {
    if constexpr (T0 == 0) {
      a = o[0];
      h = 0;
    } else {
      a += row_right<T0>(o[T0]);
      h += row_left<16 - T0>(o[T0]);
    }
    row_taps_t<TP, T0 + 1, T>(o, a, h);
  }
}

constexpr int BB = 4;    // bins of an adjoint workgroup
constexpr int ZA = 16;   // its z cells: one row of lanes per bin

template <typename T, int Q, int TP, int TY>
struct AdjointLds {
  static constexpr int ZG = ZA + TP - 1, YG = TY + TP - 1, W = TY * Q;
  size_t C, P, M, S, Sp, total;
  __host__ __device__ AdjointLds() {
    size_t o = 0;
    auto take = [&](size_t b) { size_t r = o; o = (o + b + 15) & ~(size_t)15; return r; };
    C = take((size_t)2 * YG * ZG * BB * sizeof(c2<T>));
    P = take((size_t)2 * YG * ZG * sizeof(T));
    M = take((size_t)W * Q * 8 * ZA * sizeof(T));
    S = take((size_t)W * ZG * BB * sizeof(c2<T>));
    Sp = take((size_t)W * ZG * sizeof(T));
    total = o;
  }
};

// Adjoint in the cotangent's eigenbasis: sources
//   c_k(u) = d_k conj( sum_v M_{u,v} a_k(v) )  (M the band above, both sides),
// transposed through the z and y filters onto the grid, and the primary's
// share, sum_k d_k of the same form differentiated in p.  Bins are independent
// here, so a workgroup takes four of them on a tile of TY x 16 cells: lane l
// is bin l / 16 of z cell l % 16, so that z neighbours are lane shifts within
// a row, and the point that a lane prepares the band of is l / 16 (with five
// points, the fifth on every row).  It marches along x as the forward does;
// the window holds the 2 H + 1 planes around the output plane.  The sums over
// bins of the primary's share, and its transposed z filter over points, are
// products on the matrix cores, which are otherwise idle: entry (point, shift)
// is a row of D.  Sources are added to out [cell][nbt] (zeroed by the caller:
// tiles share their halo), wm times the primary's share to direct.
// The primary's filter has PT taps from tap PO on (Daubechies-4: the node itself).
// Bound by instruction issue.  The B-spline spills: float32, 16 waves of 128 registers, 26, float64 15.
// Against the shift stencil (343 or 125 shifts per cell): 128^3, 15
// bins float32 38 -> 3.3 ms per (l, m) with the contraction apart; 32^3, 6 bins float64 0.46 -> 0.05 ms.
template <typename T, int Q, int TP, int H, int TY, int PT, int PO>
__global__ void __launch_bounds__(TY* Q * 64)
    k_band_adjoint(const c2<T>* fields, const T* prim, const T* lam_d, const T* lam_d2, T sgn, int n, int nbt, int off,
                   RuleT<T, Q, TP, H> rule, T wm, int nseg, int nchunk, c2<T>* out, T* direct) {
  using L_ = AdjointLds<T, Q, TP, TY>;
  using A4 = typename acc4<T>::type;
  constexpr int ZG = L_::ZG, YG = L_::YG, NT = TY * Q * 64, W = TY * Q, HL = TP - 1;
  constexpr int CELLS = YG * ZG, PF = (CELLS * BB + NT - 1) / NT, WIN = 2 * H + 1, PR = 3 * H + 1;
  constexpr int NP = (Q + 3) / 4;   // points whose band a lane prepares
  extern __shared__ __align__(16) char smem[];
  const L_ L;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int yc = wave / Q, sy = wave % Q;
  const int zl = lane & 15, bl = lane >> 4;
  T* Ml = reinterpret_cast<T*>(smem + L.M) + (size_t)wave * Q * 8 * ZA;
  c2<T>* S = reinterpret_cast<c2<T>*>(smem + L.S);
  T* Sp = reinterpret_cast<T*>(smem + L.Sp);
  const int mock = blockIdx.y;
  const long long n2 = (long long)n * n;
  const c2<T>* fm = fields + (long long)mock * n2 * n * nbt;
  c2<T>* om = out + (long long)mock * n2 * n * nbt;
  const T* pm = prim + (long long)mock * n2 * n;
  T* dm = direct + (long long)mock * n2 * n;
  T pz[NP][PT];   // the lane's points' primary filters
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int t = 0; t < PT; ++t) pz[i][t] = rule.p[i == 0 ? bl : 4][PO + t];
  // operand of the transposed primary filter: row t of D (float64: row 4 t, see mfma_row) is
  // sum_k p[k][t] share_k
  const int ti = std::is_same<T, double>::value ? ((zl & 3) ? PT : zl >> 2) : zl;
  T pa[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) pa[i] = ti < PT && (i == 0 || bl == 0) ? rule.p[i == 0 ? bl : 4][PO + (ti < PT ? ti : 0)] : (T)0;

  const int tz = n / ZA, ty = n / TY, seg = n / nseg, ntask = ty * tz * nseg * nchunk;
  for (int task0 = blockIdx.x; task0 < ntask; task0 += gridDim.x) {
    const int task = xcd_order(task0, ntask);
    const int chunk = task % nchunk, sg = (task / nchunk) % nseg, tile = task / (nchunk * nseg);
    const int b0 = chunk * BB, nbc = nbt - b0 < BB ? nbt - b0 : BB;
    const int y0 = (tile / tz) * TY + off, z0 = (tile % tz) * ZA + off, x0 = sg * seg;
    // eigenvalues of the real and the imaginary part (a pair item's parts are two multipoles' real fields,
    // whose sources carry no conjugate: sgn = 1, else -1)
    const T dk = bl < nbc ? lam_d[(long long)mock * nbt + b0 + bl] : (T)0;
    const T dk2 = bl < nbc ? lam_d2[(long long)mock * nbt + b0 + bl] : (T)0;
    int src[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int e = tid + i * NT, bb = e % BB, cell = e / BB;
      const int yy = wrap_n(y0 + cell / ZG, n), zz = wrap_n(z0 + cell % ZG, n);
      src[i] = cell < CELLS ? (yy * n + zz) * nbt + b0 + (bb < nbc ? bb : 0) : -1;
    }
    int psrc = -1;
    if (tid < CELLS) psrc = wrap_n(y0 + tid / ZG, n) * n + wrap_n(z0 + tid % ZG, n);
    c2<T> win[WIN][Q];
    T pr[NP][PR], dp[NP][2 * H + 1];   // primary at planes u - H .. u + 2 H; its share at u - H .. u + H
#pragma unroll
    for (int i = 0; i < WIN; ++i)
#pragma unroll
      for (int s = 0; s < Q; ++s) win[i][s] = mk<T>(0, 0);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
#pragma unroll
      for (int j = 0; j < PR; ++j) pr[i][j] = 0;
#pragma unroll
      for (int j = 0; j <= 2 * H; ++j) dp[i][j] = 0;
    }
    c2<T> nextc[PF];
    T nextp = 0;
    auto fetch = [&](int x) {   // fields of plane x, primary of plane x + H
      const c2<T>* fp = fm + (long long)wrap_n(x, n) * n2 * nbt;
#pragma unroll
      for (int i = 0; i < PF; ++i) nextc[i] = src[i] >= 0 ? fp[src[i]] : mk<T>(0, 0);
      if (psrc >= 0) nextp = pm[(long long)wrap_n(x + H, n) * n2 + psrc];
    };
    fetch(x0 - 2 * H);
    // planes X = x0 - 2 H + st, output plane u = X - H: H planes that fill the primary's window, 2 H the
    // fields', seg with output, 2 H that drain the primary's share
    const int steps = 5 * H + seg;
    for (int st0 = 0; st0 < steps; st0 += WIN) {
#pragma unroll
      for (int u = 0; u < WIN; ++u) {
        const int st = st0 + u, X = x0 - 2 * H + st;
        if (st < steps) {
          // keep the lane's LDS addresses inside the step: hoisted out of the loop they would pin registers
          int z = zl, b = bl;
          asm volatile("" : "+v"(z), "+v"(b));
          const int zh = z < HL ? 16 + z : 16;   // the halo cell of the first lanes of a row
          const bool have_f = st >= H && st < 3 * H + seg;
          const bool have_o = st >= 3 * H && st < 3 * H + seg;
          c2<T>* C = reinterpret_cast<c2<T>*>(smem + L.C) + (size_t)(st & 1) * CELLS * BB;
          T* P = reinterpret_cast<T*>(smem + L.P) + (st & 1) * CELLS;
#pragma unroll
          for (int i = 0; i < PF; ++i)
            if (src[i] >= 0) C[tid + i * NT] = nextc[i];
          if (psrc >= 0) P[tid] = nextp;
          __syncthreads();
          if (st + 1 < 3 * H + seg) fetch(X + 1);
          // primary: y filter, z neighbours, z filter of the lane's points
          {
            T a = 0, h = 0, v[PO + PT];
#pragma unroll
            for (int t = 0; t < PT; ++t) {
              const T w = rule.p[sy][PO + t];
              a += w * P[(yc + PO + t) * ZG + z];
              h += w * P[(yc + PO + t) * ZG + zh];
            }
            row_taps<PO + PT, 0, T>(a, h, v);
#pragma unroll
            for (int i = 0; i < NP; ++i) {
#pragma unroll
              for (int j = 0; j + 1 < PR; ++j) pr[i][j] = pr[i][j + 1];
              T p = 0;
#pragma unroll
              for (int t = 0; t < PT; ++t) p += pz[i][t] * v[PO + t];
              pr[i][PR - 1] = p;
            }
          }
          // fields: y filter, z neighbours, z filter
          if (have_f) {
            c2<T> a = mk<T>(0, 0), h = mk<T>(0, 0);
#pragma unroll
            for (int t = 0; t < TP; ++t) {
              const T w = rule.f[sy][t];
              const c2<T> va = C[((yc + t) * ZG + z) * BB + b], vh = C[((yc + t) * ZG + zh) * BB + b];
              a.x += w * va.x;
              a.y += w * va.y;
              h.x += w * vh.x;
              h.y += w * vh.y;
            }
            T vx[TP], vy[TP];
            row_taps<TP, 0, T>(a.x, h.x, vx);
            row_taps<TP, 0, T>(a.y, h.y, vy);
#pragma unroll
            for (int s = 0; s < Q; ++s) {
              c2<T> f = mk<T>(0, 0);
#pragma unroll
              for (int t = 0; t < TP; ++t) {
                f.x += rule.f[s][t] * vx[t];
                f.y += rule.f[s][t] * vy[t];
              }
              win[u][s] = f;
            }
          }
          A4 qd[NP];
#pragma unroll
          for (int i = 0; i < NP; ++i) qd[i] = A4{0, 0, 0, 0};
          if (have_o) {
            // M_d(u) and M_d(u + d) of the lane's points, to the wave's rows [point][0 | 4 + d][z]
#pragma unroll
            for (int i = 0; i < NP; ++i) {
              T m[8];
#pragma unroll
              for (int d = 0; d < 4; ++d) m[d] = m[4 + d] = 0;
#pragma unroll
              for (int d = 0; d <= H; ++d)
#pragma unroll
                for (int j = 0; j <= 2 * H - d; ++j) {   // offsets j - H <= H - d: the rest vanish
                  m[d] += rule.g[d][j] * pr[i][j];
                  if (d > 0) m[4 + d] += rule.g[d][j] * pr[i][j + d];
                }
              const int s = i == 0 ? b : 4;
              T* row = Ml + (size_t)s * 8 * ZA + 4 * z;
#pragma unroll
              for (int d = 0; d < 4; ++d) {
                row[d] = m[d];
                row[4 * ZA + d] = m[4 + d];
              }
            }
            col_sync<true>();
            T ox[TP], oy[TP];
#pragma unroll
            for (int t = 0; t < TP; ++t) ox[t] = oy[t] = 0;
#pragma unroll
            for (int s = 0; s < Q; ++s) {
              __builtin_amdgcn_sched_barrier(0);   // one point's coefficients in registers at a time
              T m[4], mu[4];
              const T* row = Ml + (size_t)s * 8 * ZA + 4 * z;
#pragma unroll
              for (int d = 0; d < 4; ++d) {
                m[d] = row[d];
                mu[d] = row[4 * ZA + d];
              }
              const c2<T> f = win[(u + WIN - H) % WIN][s];
              T hx = m[0] * f.x, hy = m[0] * f.y;
              T q[H + 1];
              const T fx = dk * f.x, fy = dk2 * f.y;
              q[0] = fx * f.x + fy * f.y;
#pragma unroll
              for (int d = 1; d <= H; ++d) {
                const c2<T> lo = win[(u + 2 * WIN - H - d) % WIN][s], hi = win[(u + WIN - H + d) % WIN][s];
                hx += m[d] * lo.x + mu[d] * hi.x;
                hy += m[d] * lo.y + mu[d] * hi.y;
                q[d] = fx * lo.x + fy * lo.y;
              }
#pragma unroll
              for (int t = 0; t < TP; ++t) {
                ox[t] += rule.f[s][t] * hx;
                oy[t] += rule.f[s][t] * hy;
              }
              // sums over bins: entry (point, shift) is the row of D that the lane row of that point reads
#pragma unroll
              for (int d = 0; d <= H; ++d) {
                const int row4 = std::is_same<T, double>::value ? 4 * d + (s & 3) : 4 * (s & 3) + d;
                if (s < 4) {
                  qd[0] = mfma16(z == row4 ? (T)1 : (T)0, q[d], qd[0]);
                } else {   // the fifth point, on every lane row
                  const bool mine = std::is_same<T, double>::value ? (z >> 2) == d : (z & 3) == d;
                  qd[NP - 1] = mfma16(mine ? (T)1 : (T)0, q[d], qd[NP - 1]);
                }
              }
            }
            T ax, hx, ay, hy;
            row_taps_t<TP, 0, T>(ox, ax, hx);
            row_taps_t<TP, 0, T>(oy, ay, hy);
            S[(wave * ZG + z) * BB + b] = mk<T>(dk * ax, sgn * (dk2 * ay));
            if (z < HL) S[(wave * ZG + 16 + z) * BB + b] = mk<T>(dk * hx, sgn * (dk2 * hy));
          }
          // the primary's share at plane u - H is complete with plane u
          if (st >= 3 * H) {
            A4 op = A4{0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < NP; ++i) {
#pragma unroll
              for (int j = 0; j <= 2 * H; ++j) {
                T a = dp[i][j] + rule.g[0][j] * qd[i][0];
#pragma unroll
                for (int d = 1; d <= H; ++d)
                  if (j <= 2 * H - d) a += ((T)2 * rule.g[d][j]) * qd[i][d];
                dp[i][j] = a;
              }
              op = mfma16(pa[i], dp[i][0], op);
#pragma unroll
              for (int j = 0; j < 2 * H; ++j) dp[i][j] = dp[i][j + 1];
              dp[i][2 * H] = 0;
            }
            T o[PO + PT], a, h;
#pragma unroll
            for (int t = 0; t < PO; ++t) o[t] = 0;
#pragma unroll
            for (int t = 0; t < PT; ++t) o[PO + t] = op[t];
            row_taps_t<PO + PT, 0, T>(o, a, h);
            if (b == 0) {
              Sp[wave * ZG + z] = a;
              if (z < HL) Sp[wave * ZG + 16 + z] = h;
            }
            __syncthreads();
          }
          // transposed y filter, a grid row yg per two waves, added to the grid
          if (have_o) {
            const long long xo = (long long)wrap_n(X - H, n) * n2;
            for (int r = wave; r < 2 * YG; r += W) {
              const int le = 16 * b + z, yg = r >> 1, zg = (r & 1) ? 16 + (le >> 2) : le >> 2, bb = le & 3;
              if (zg < ZG) {
                c2<T> a = mk<T>(0, 0);
#pragma unroll
                for (int t = 0; t < TP; ++t) {
                  const int y = yg - t;
                  if (y >= 0 && y < TY) {
#pragma unroll
                    for (int s = 0; s < Q; ++s) {
                      const c2<T> v = S[((y * Q + s) * ZG + zg) * BB + bb];
                      a.x += rule.f[s][t] * v.x;
                      a.y += rule.f[s][t] * v.y;
                    }
                  }
                }
                if (bb < nbc) {
                  T* dst = reinterpret_cast<T*>(om + (xo + (long long)wrap_n(y0 + yg, n) * n + wrap_n(z0 + zg, n)) * nbt +
                                                b0 + bb);
                  unsafeAtomicAdd(dst, a.x);
                  unsafeAtomicAdd(dst + 1, a.y);
                }
              }
            }
          }
          if (st >= 3 * H) {
            const long long xo = (long long)wrap_n(X - 2 * H, n) * n2;
            // the last threads first: the first waves may still be at the sources
            for (int e = NT - 1 - tid; e < CELLS; e += NT) {
              const int yg = e / ZG, zg = e % ZG;
              T a = 0;
#pragma unroll
              for (int t = PO; t < PO + PT; ++t) {
                const int y = yg - t;
                if (y >= 0 && y < TY) {
#pragma unroll
                  for (int s = 0; s < Q; ++s) a += rule.p[s][t] * Sp[(y * Q + s) * ZG + zg];
                }
              }
              unsafeAtomicAdd(dm + xo + (long long)wrap_n(y0 + yg, n) * n + wrap_n(z0 + zg, n), wm * a);
            }
          }
        }
      }
    }
    __syncthreads();   // the next task refills the planes and the sums
  }
}

template <typename K> hipError_t allow_band_lds(K kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

// segments of the march: enough workgroups for the 256 CUs (two each, and a
// second round), while a segment stays long against the 2 H (forward) or
// 5 H (adjoint) extra planes that it costs
int band_segments(int n, long long tiles, int batch) {
  int s = 1;
  while (n / (2 * s) >= 16 && tiles * batch * s < 1024) s *= 2;
  while (n / (2 * s) >= 8 && tiles * batch * s < 256) s *= 2;
  return s;
}

// rows of cells of a forward workgroup (TY), by registers: 16 waves (TY = 4, 128 registers) hold the float32
// B-spline with up to 16 bins; two bin halves spill there (256^3, 20 bins: 19.2 ms against 17.8 ms
// with 8 waves), as do float64 and the five points of Daubechies-4
int contract_rows(int prec, int q, int nl) {
  if (q == 4) return !prec && nl <= 16 ? 4 : 2;
  return prec && nl > 16 ? 1 : 2;
}

template <typename T, int Q, int TP, int H, int TY, int NH>
hipError_t contract_t(const void* fields, const void* prim, int n, const BinPair& bp, const BandRule& rule,
                      double* partials, int nwg, bool pair, int batch, hipStream_t st) {
  const int nl = bp.na + bp.nc;
  if (contract_rows(sizeof(T) == 8, Q, nl) != TY) return hipErrorInvalidValue;
  const size_t lds = ContractLds<T, Q, TP, TY, NH>(nl).total;
  auto kern = k_band_contract<T, Q, TP, H, TY, NH>;
  hipError_t e = allow_band_lds(kern, lds);
  if (e != hipSuccess) return e;
  const int nseg = band_segments(n, (long long)(n / TY) * (n / 4), batch);
  kern<<<dim3(nwg, batch), TY * Q * 64, lds, st>>>(static_cast<const c2<T>*>(fields), static_cast<const T*>(prim), n,
                                                  bp.nbt, bp.a0, bp.na, bp.c0, nl, rule.off,
                                                  rule_of<T, Q, TP, H>(rule), nseg, pair ? 1 : 0, partials);
  return hipGetLastError();
}

template <typename T, int Q, int TP, int H, int TY, int PT, int PO>
hipError_t adjoint_t(const void* fields, const void* prim, const void* lam_d, const void* lam_d2, int n, int nbt, const BandRule& rule,
                     double wm, int batch, void* out, void* direct, hipStream_t st) {
  const size_t lds = AdjointLds<T, Q, TP, TY>().total;
  auto kern = k_band_adjoint<T, Q, TP, H, TY, PT, PO>;
  hipError_t e = allow_band_lds(kern, lds);
  if (e != hipSuccess) return e;
  const int nchunk = (nbt + BB - 1) / BB;
  const long long tiles = (long long)(n / TY) * (n / ZA) * nchunk;
  const int nseg = band_segments(n, tiles, batch);
  const long long tasks = tiles * nseg;
  kern<<<dim3((unsigned)(tasks < 65536 ? tasks : 65536), batch), TY * Q * 64, lds, st>>>(
      static_cast<const c2<T>*>(fields), static_cast<const T*>(prim), static_cast<const T*>(lam_d),
      static_cast<const T*>(lam_d2 ? lam_d2 : lam_d), lam_d2 ? (T)1 : (T)-1, n, nbt, rule.off,
      rule_of<T, Q, TP, H>(rule), (T)wm, nseg, nchunk, static_cast<c2<T>*>(out), static_cast<T*>(direct));
  return hipGetLastError();
}

}  // namespace

int band_contract_tasks(int prec, int n, int nl, const BandRule& rule, int batch) {
  const int tiles = (n / contract_rows(prec, rule.q, nl)) * (n / 4);
  return tiles * band_segments(n, tiles, batch);
}

hipError_t launch_band_contract(int prec, const void* fields, const void* prim, int n, const BinPair& bp,
                                const BandRule& rule, double* partials, int nwg, bool pair, int batch, hipStream_t st) {
  const int nl = bp.na + bp.nc;
  if (nl > kBandBins || n % 4) return hipErrorInvalidValue;
  const bool two = nl > 16;
  if (rule.q == 4) {
    if (prec) {
      return two ? contract_t<double, 4, 4, 3, 2, 2>(fields, prim, n, bp, rule, partials, nwg, pair, batch, st)
                 : contract_t<double, 4, 4, 3, 2, 1>(fields, prim, n, bp, rule, partials, nwg, pair, batch, st);
    }
    return two ? contract_t<float, 4, 4, 3, 2, 2>(fields, prim, n, bp, rule, partials, nwg, pair, batch, st)
               : contract_t<float, 4, 4, 3, 4, 1>(fields, prim, n, bp, rule, partials, nwg, pair, batch, st);
  }
  if (rule.q != 5) return hipErrorInvalidValue;
  if (prec) {
    return two ? contract_t<double, 5, 5, 2, 1, 2>(fields, prim, n, bp, rule, partials, nwg, pair, batch, st)
               : contract_t<double, 5, 5, 2, 2, 1>(fields, prim, n, bp, rule, partials, nwg, pair, batch, st);
  }
  return two ? contract_t<float, 5, 5, 2, 2, 2>(fields, prim, n, bp, rule, partials, nwg, pair, batch, st)
             : contract_t<float, 5, 5, 2, 2, 1>(fields, prim, n, bp, rule, partials, nwg, pair, batch, st);
}

hipError_t launch_band_adjoint(int prec, const void* fields, const void* prim, const void* lam_d, const void* lam_d2, int n, int nbt,
                               const BandRule& rule, double wm, int batch, void* out, void* direct, hipStream_t st) {
  if (n % ZA) return hipErrorInvalidValue;
#define BAND_ADJ(...) adjoint_t<__VA_ARGS__>(fields, prim, lam_d, lam_d2, n, nbt, rule, wm, batch, out, direct, st)
  if (rule.q == 4) return prec ? BAND_ADJ(double, 4, 4, 3, 2, 4, 0) : BAND_ADJ(float, 4, 4, 3, 4, 4, 0);
  if (rule.q != 5) return hipErrorInvalidValue;
  return prec ? BAND_ADJ(double, 5, 5, 2, 1, 1, 2) : BAND_ADJ(float, 5, 5, 2, 2, 1, 2);
#undef BAND_ADJ
}

}  // namespace mp3

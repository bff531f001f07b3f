// scatter.hip -- adjoint sources of the particle summation onto the grid.
#include "fft_core.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

#include <hip/hip_runtime.h>

namespace mp3 {

namespace {

constexpr int ST = 8;              // owner tile side (nodes)
constexpr int SB = ST + 3;         // first-tap positions per axis that reach the tile
constexpr int SKEYS = SB * SB;     // (x, y) buckets of the stage
constexpr int SNT = 512;           // threads: wave w owns the tile's x plane w
constexpr int SR = 6;              // source elements of a thread in flight
template <typename T> constexpr int stage_q() { return sizeof(T) == 4 ? 256 : 128; }   // particles of a stage

template <typename T> __device__ __forceinline__ void load4(const T* p, T* o);
template <> __device__ __forceinline__ void load4<float>(const float* p, float* o) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
}
template <> __device__ __forceinline__ void load4<double>(const double* p, double* o) {
  const double2 u = *reinterpret_cast<const double2*>(p), v = *reinterpret_cast<const double2*>(p + 2);
  o[0] = u.x; o[1] = u.y; o[2] = v.x; o[3] = v.y;
}

// the value of the other lane of a pair
__device__ __forceinline__ float swap_pair(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xb1, 0xf, 0xf, true));
}
__device__ __forceinline__ double swap_pair(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0xb1, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0xb1, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

template <typename T>
struct ScatterLds {
  size_t src, wt, id, key, sid, start, total;
  __host__ __device__ ScatterLds(int nbc) {
    constexpr int Q = stage_q<T>();
    size_t o = 0;
    auto take = [&](size_t b) { size_t r = o; o = (o + b + 15) & ~(size_t)15; return r; };
    src = take((size_t)Q * 2 * nbc * sizeof(T));
    wt = take((size_t)Q * 3 * ST * sizeof(T));
    id = take((size_t)(Q + SNT) * sizeof(int));
    key = take((size_t)(Q + SNT) * sizeof(int));
    sid = take((size_t)Q * sizeof(int));
    start = take((size_t)(SKEYS + 1) * sizeof(int));
    total = o;
  }
};

// c_b(x) = sum_i phi(u_i - x) s_b(i), by pulling: a workgroup owns an 8^3-node
// tile and writes it once (no atomics).  Candidates are the particles of the
// 4^3-cell sort tiles covering cells x0 - 4 .. x0 + 11 per axis; those whose
// stencil reaches the tile are staged up to Q at a time in LDS, ordered by the
// (x, y) of their first tap, with their sources and their tap weights spread
// over the tile's eight nodes per axis (zero off the stencil).  The sum is then
// a product on the matrix cores: D[node][column] += W[node][particle]
// s[particle][column], 16 nodes (two y, eight z at the wave's x), four
// particles and 16 of the 2 nbc real columns per instruction.  A row block takes the
// particles of 4 x 5 of the 11 x 11 buckets, four contiguous runs of the
// stage, so that a sixth of the stage is multiplied rather than all of it: a particle's four y taps
// meet 2 or 3 row blocks, so that 4 x 2.5 x 16 / 64 = 2.5 products are spent per tap, with no divergence.
// (float64: 112 bytes of scratch a thread.)
// Bound by the matrix loop (16 ms of 30 at 512^3: operand addresses and matrix
// products share the issue slots) and the staging (8 ms).  Against one thread
// per node walking its buckets, where a wave waits for the longest: 512^3, 5e7
// particles, 20 bins float32 75.6 -> 30.2 ms per launch; 128^3, 1e6 particles, 15 bins 1.51 -> 0.61 ms.
template <typename T, int CB>
__global__ void __launch_bounds__(SNT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2))) k_scatter_source(const int* tcell, const T* twt, const int* toff, const T* src,
                                                        int n, int nbins, int nchunk, int bpc, T* out) {
  constexpr int Q = stage_q<T>();
  using A4 = typename acc4<T>::type;
  extern __shared__ __align__(16) char smem[];
  __shared__ int pre[65];
  __shared__ int cbase[64];
  __shared__ int qn;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mock = blockIdx.y / nchunk, b0 = (blockIdx.y % nchunk) * bpc;
  const int nbc = min(bpc, nbins - b0), ncol = 2 * nbc;
  const ScatterLds<T> L(bpc);
  T* ssrc = reinterpret_cast<T*>(smem + L.src);
  T* swt = reinterpret_cast<T*>(smem + L.wt);
  int* qid = reinterpret_cast<int*>(smem + L.id);
  int* qkey = reinterpret_cast<int*>(smem + L.key);     // x | y << 4 | z << 8, first tap + 3
  int* sid = reinterpret_cast<int*>(smem + L.sid);      // particle of a slot
  int* start = reinterpret_cast<int*>(smem + L.start);
  const int no = n / ST;
  const int ot = xcd_order(blockIdx.x, no * no * no);
  const int oi[3] = {ot / (no * no), (ot / no) % no, ot % no};
  const int ntd = n / 4;
  if (tid < 64) {
    const int sx = (2 * oi[0] - 1 + tid / 16 + ntd) % ntd, sy = (2 * oi[1] - 1 + (tid / 4) % 4 + ntd) % ntd;
    const int sz = (2 * oi[2] - 1 + tid % 4 + ntd) % ntd;
    const long long tile = ((long long)mock * ntd + sx) * ntd * ntd + (long long)sy * ntd + sz;
    const int a = toff[tile];
    cbase[tid] = a;
    int c = toff[tile + 1] - a, incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (tid >= o) incl += v;
    }
    pre[tid + 1] = incl;
    if (tid == 0) {
      pre[0] = 0;
      qn = 0;
    }
  }
  __syncthreads();
  const int total = pre[64];
  // operand positions of the lane: node (yy, z) of a row block, particle kk of four, column j
  const int yy = (lane >> 3) & 1, z = lane & 7, kk = lane >> 4, j = lane & 15;
  const T* wrow = swt;
  const int wyo = ST + yy, wzo = 2 * ST + z;
  int col[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c) col[c] = 16 * c + j < ncol ? 16 * c + j : 0;   // absent columns are not written
  A4 acc[4][CB];
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[y][c] = A4{0, 0, 0, 0};

  // candidate t of the tile: its sorted index and packed cell (-1: none)
  auto candidate = [&](int t, int& k) {
    k = 0;
    if (t >= total) return -1;
    int lo = 0, hi = 64;                      // pre[lo] <= t < pre[hi]
#pragma unroll
    for (int it = 0; it < 6; ++it) {
      const int mid = (lo + hi) >> 1;
      if (pre[mid] <= t) lo = mid; else hi = mid;
    }
    k = cbase[lo] + (t - pre[lo]);
    return tcell[k];
  };
  int knext = 0, cnext = candidate(tid, knext);
  for (int t0 = 0; t0 < total; t0 += SNT) {
    // candidates that reach the tile, appended to the list; the next ones' cells are in flight meanwhile
    const int k = knext, cell = cnext;
    cnext = candidate(t0 + SNT + tid, knext);
    const int cb[3] = {(cell & 1023) - 1, ((cell >> 10) & 1023) - 1, (cell >> 20) - 1};   // first tap per axis
    bool reach = cell >= 0;
    int key = 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int r = (cb[d] - ST * oi[d] + 3) & (n - 1);   // 0 .. 10 when the stencil reaches the tile
      reach = reach && r < SB;
      key |= r << (4 * d);
    }
    const unsigned long long m = __ballot(reach);
    int at = 0;
    if (lane == 0 && m) at = atomicAdd(&qn, __popcll(m));
    at = __shfl(at, 0, 64);
    if (reach) {
      const int q = at + __popcll(m & ((1ull << lane) - 1));
      qid[q] = k;
      qkey[q] = key;
    }
    __syncthreads();
    const bool last = t0 + SNT >= total;
    int nq = qn;
    __syncthreads();   // every thread has read qn before the next candidates are appended
    // a stage whenever the list may overflow with the next candidates, and at the end
    while (nq >= Q || (last && nq > 0)) {
      const int ns = nq < Q ? nq : Q;
      // weights of particle tid in flight while the slots in (x, y) order are found
      T w[12];
      int my = 0, mykey = 0, kq = 0, id = 0;
      for (int c = tid; c <= SKEYS; c += SNT) start[c] = 0;
      if (tid < ns) {
        id = qid[tid];
        kq = qkey[tid];
        const T* wr = twt + (long long)id * 12;
#pragma unroll
        for (int e = 0; e < 12; e += 4) load4<T>(wr + e, w + e);
        mykey = (kq & 15) * SB + ((kq >> 4) & 15);
      }
      __syncthreads();
      if (tid < ns) my = atomicAdd(&start[mykey + 1], 1);   // rank within the bucket
      __syncthreads();
      if (tid < 64) {   // inclusive sums of the SKEYS + 1 = 122 counts, two per lane
        const int c0 = start[2 * tid < SKEYS + 1 ? 2 * tid : 0], c1 = start[2 * tid + 1 < SKEYS + 1 ? 2 * tid + 1 : 0];
        int incl = c0 + c1;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int v = __shfl_up(incl, o, 64);
          if (tid >= o) incl += v;
        }
        if (2 * tid < SKEYS + 1) start[2 * tid] = incl - c1;
        if (2 * tid + 1 < SKEYS + 1) start[2 * tid + 1] = incl;
      }
      __syncthreads();
      if (tid < ns) {
        const int s = start[mykey] + my;
        sid[s] = id;
        T* row = swt + (size_t)s * 3 * ST;
#pragma unroll
        for (int e = 0; e < 3 * ST; ++e) row[e] = 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const int r = ((kq >> (4 * d)) & 15) - 3;   // first tap's node
#pragma unroll
          for (int a = 0; a < 4; ++a)
            if ((unsigned)(r + a) < (unsigned)ST) row[d * ST + r + a] = w[4 * d + a];
        }
      }
      __syncthreads();
      // sources of the stage in slot order, SR elements of a thread in flight
      {
        const int count = ns * nbc, ds = SNT / nbc, db = SNT % nbc;
        int s = tid / nbc, b = tid % nbc;
        for (int e0 = tid; e0 < count; e0 += SR * SNT) {
          c2<T> v[SR];
#pragma unroll
          for (int i = 0; i < SR; ++i) {
            if (e0 + i * SNT < count) v[i] = reinterpret_cast<const c2<T>*>(src)[(long long)sid[s] * nbins + b0 + b];
            s += ds;
            b += db;
            if (b >= nbc) {
              b -= nbc;
              ++s;
            }
          }
#pragma unroll
          for (int i = 0; i < SR; ++i)
            if (e0 + i * SNT < count) reinterpret_cast<c2<T>*>(ssrc)[e0 + i * SNT] = v[i];
        }
      }
      // runs of the wave's x plane: bucket rows x .. x + 3, per pair of y
      int bound = 0;
      if (lane < 32) bound = start[(wave + ((lane >> 1) & 3)) * SB + 2 * (lane >> 3) + 5 * (lane & 1)];
      __syncthreads();
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        // the four runs as one list: element i is slot i + o0, o1, o2 or o3 by the running lengths
        const int a0 = __builtin_amdgcn_readlane(bound, 8 * y), e0 = __builtin_amdgcn_readlane(bound, 8 * y + 1);
        const int a1 = __builtin_amdgcn_readlane(bound, 8 * y + 2), e1 = __builtin_amdgcn_readlane(bound, 8 * y + 3);
        const int a2 = __builtin_amdgcn_readlane(bound, 8 * y + 4), e2 = __builtin_amdgcn_readlane(bound, 8 * y + 5);
        const int a3 = __builtin_amdgcn_readlane(bound, 8 * y + 6), e3 = __builtin_amdgcn_readlane(bound, 8 * y + 7);
        const int l1 = e0 - a0, l2 = l1 + e1 - a1, l3 = l2 + e2 - a2, l4 = l3 + e3 - a3;
        const int o1 = a1 - l1, o2 = a2 - l2, o3 = a3 - l3;
        // two groups of four particles at a time: the operands of both are in flight together
        for (int s = 0; s < l4; s += 8) {
          T a[2], v[2][CB];
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            const int i = min(s + 4 * g + kk, l4 - 1);
            int o = a0;
            o = i >= l1 ? o1 : o;
            o = i >= l2 ? o2 : o;
            o = i >= l3 ? o3 : o;
            const int p = i + o;
            const T* w = wrow + __umul24(p, 3 * ST);
            a[g] = w[wave] * w[wyo + 2 * y] * w[wzo];
            const T* sp = ssrc + __umul24(p, ncol);
#pragma unroll
            for (int c = 0; c < CB; ++c) v[g][c] = sp[col[c]];
          }
          a[0] = s + kk < l4 ? a[0] : (T)0;
          a[1] = s + 4 + kk < l4 ? a[1] : (T)0;
#pragma unroll
          for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int c = 0; c < CB; ++c) acc[y][c] = mfma16(a[g], v[g][c], acc[y][c]);
        }
      }
      __syncthreads();
      // what did not fit moves to the front of the list
      const int rest = nq - ns;
      int ri = 0, rk = 0;
      if (tid < rest) {
        ri = qid[ns + tid];
        rk = qkey[ns + tid];
      }
      __syncthreads();
      if (tid < rest) {
        qid[tid] = ri;
        qkey[tid] = rk;
      }
      if (tid == 0) qn = rest;
      nq = rest;
      __syncthreads();
    }
  }
  // rows of D are (yy, z), columns (bin, re / im): neighbouring lanes exchange parts, so that each
  // writes whole complex values, 16 bytes of a bin's run of eight z
  const long long n3 = (long long)n * n * n;
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const bool odd = j & 1;
      const A4 a = acc[y][c];
      const T r0 = swap_pair(odd ? a[0] : a[2]), r1 = swap_pair(odd ? a[1] : a[3]);
      const int b = b0 + 8 * c + (j >> 1);
      T* o = out + (((long long)mock * nbins + b) * n3 + ((long long)(ST * oi[0] + wave) * n + ST * oi[1] + 2 * y) * n +
                    ST * oi[2]) * 2;
      if (16 * c + j < ncol) {
        if constexpr (sizeof(T) == 4) {   // rows 4 (l / 16) + i: two z of one y
          T* p = o + 2 * ((long long)(lane >> 5) * n + 4 * ((lane >> 4) & 1) + (odd ? 2 : 0));
          *reinterpret_cast<float4*>(p) = odd ? make_float4(r0, a[2], r1, a[3]) : make_float4(a[0], r0, a[1], r1);
        } else {                          // rows 4 i + l / 16: two z of y = odd
          T* p = o + 2 * ((long long)(odd ? n : 0) + (lane >> 4));
          *reinterpret_cast<double2*>(p) = odd ? make_double2(r0, a[2]) : make_double2(a[0], r0);
          *reinterpret_cast<double2*>(p + 8) = odd ? make_double2(r1, a[3]) : make_double2(a[1], r1);
        }
      }
    }
}

template <typename T, int CB>
hipError_t scatter_cb(const int* tcell, const void* twt, const int* toff, const void* src, int n, int nbins, int nchunk,
                      int bpc, int batch, void* out, hipStream_t st) {
  const size_t lds = ScatterLds<T>(bpc).total;
  auto kern = k_scatter_source<T, CB>;
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const int no = n / ST;
  kern<<<dim3(no * no * no, batch * nchunk), SNT, lds, st>>>(tcell, static_cast<const T*>(twt), toff,
                                                            static_cast<const T*>(src), n, nbins, nchunk, bpc,
                                                            static_cast<T*>(out));
  return hipGetLastError();
}

template <typename T>
hipError_t scatter_t(const int* tcell, const void* twt, const int* toff, const void* src, int n, int nbins, int batch,
                     void* out, hipStream_t st) {
  // at most 24 bins (three column blocks) a pass, split evenly
  const int nchunk = (nbins + 23) / 24, bpc = (nbins + nchunk - 1) / nchunk;
  const int cb = (2 * bpc + 15) / 16;
  if (cb == 1) return scatter_cb<T, 1>(tcell, twt, toff, src, n, nbins, nchunk, bpc, batch, out, st);
  if (cb == 2) return scatter_cb<T, 2>(tcell, twt, toff, src, n, nbins, nchunk, bpc, batch, out, st);
  return scatter_cb<T, 3>(tcell, twt, toff, src, n, nbins, nchunk, bpc, batch, out, st);
}

}  // namespace

hipError_t launch_scatter_source(int prec, const int* tcell, const void* twt, const int* toff, const void* src, int n,
                                 int nbins, int batch, void* out, hipStream_t st) {
  return prec ? scatter_t<double>(tcell, twt, toff, src, n, nbins, batch, out, st)
              : scatter_t<float>(tcell, twt, toff, src, n, nbins, batch, out, st);
}

}  // namespace mp3

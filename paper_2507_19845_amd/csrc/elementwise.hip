// HBM-bound kernels of the stage: LayerNorm forward/backward (with the residual
// gradient and the bias gradient of the preceding linear layer folded in), column sums
// for the other bias gradients, and the fixed-order reduction of per-workgroup partial
// sums.  A token row belongs to one wave where it fits its registers (then without a barrier), else to
// a whole workgroup; 16-byte loads, the row cached in registers, fp32 statistics.
#include "../../include/gpt_stage.h"

#include <mutex>

#include "reduce.hpp"

namespace gpts {

constexpr int kLnThreads = 256;

// 8 consecutive elements <-> fp32 registers (one 16-byte access for bf16, two for fp32)
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
  for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
}
__device__ __forceinline__ void load8(const bf16* p, float (&v)[8]) {
  const bf16x8 a = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (float)a[e];
}
__device__ __forceinline__ void load8(const f16* p, float (&v)[8]) {
  const f16x8 a = *reinterpret_cast<const f16x8*>(p);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (float)a[e];
}
__device__ __forceinline__ void store8(f16* p, const float (&v)[8]) {
  f16x8 a;
#pragma unroll
  for (int e = 0; e < 8; ++e) a[e] = sat_f16(v[e]);
  *reinterpret_cast<f16x8*>(p) = a;
}
__device__ __forceinline__ void store8(float* p, const float (&v)[8]) {
  f32x4 a, b;
#pragma unroll
  for (int e = 0; e < 4; ++e) { a[e] = v[e]; b[e] = v[4 + e]; }
  *reinterpret_cast<f32x4*>(p) = a;
  *reinterpret_cast<f32x4*>(p + 4) = b;
}
__device__ __forceinline__ void store8(bf16* p, const float (&v)[8]) {
  bf16x8 a;
#pragma unroll
  for (int e = 0; e < 8; ++e) a[e] = (bf16)v[e];
  *reinterpret_cast<bf16x8*>(p) = a;
}

typedef int i32x4 __attribute__((ext_vector_type(4)));
// 8 consecutive elements kept as they are stored (half the registers for 16-bit types)
template <typename T> struct Raw8 {
  typedef T v8 __attribute__((ext_vector_type(8)));
  v8 v;
  __device__ __forceinline__ void load(const T* p) { v = *reinterpret_cast<const v8*>(p); }
  __device__ __forceinline__ float get(int e) const { return (float)v[e]; }
  // the compiler takes the registers as written: nothing derived from them is kept across this
  __device__ __forceinline__ void opaque() {
    i32x4 r = __builtin_bit_cast(i32x4, v);
    asm volatile("" : "+v"(r));
    v = __builtin_bit_cast(v8, r);
  }
};
template <> struct Raw8<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const f32x4*>(p);
    b = *reinterpret_cast<const f32x4*>(p + 4);
  }
  __device__ __forceinline__ float get(int e) const { return e < 4 ? a[e] : b[e - 4]; }
  __device__ __forceinline__ void opaque() { asm volatile("" : "+v"(a), "+v"(b)); }
};

// ----------------------------------------------------------------- LN fwd ----
// Per token: mu = mean(x), var = mean((x-mu)^2), r = 1/sqrt(var+eps),
// out = (x-mu) r gamma + beta.  TX = type of x (the residual stream, fp32 inside
// bf16 stages), T = type of gamma/beta, TO = type of out (T, or fp16 when the forward
// activations of a bf16 stage are kept in fp16).  RW = waves per row (1: four rows per
// workgroup, no barrier; 4), NCH = 8-element chunks per lane.  xcopy (may be null): x as fp32, the
// first layer's own copy of the stage input.
// Bound by HBM from some thousand rows on, by launch and latency below.  With a wave per row instead of a
// workgroup, whose threads were half idle: 8192 rows of 512 9.7 -> 7.4 us, of 768 10.9 -> 7.7 us,
// 3968 of 2048 9.7 -> 8.7 us.
// blockIdx.y: the micro-batch; strides between them in units of 16 bytes
template <typename P> __device__ __forceinline__ P* at_mb(P* p, uint32_t stride16, uint32_t mb) {
  return (P*)((const char*)p + (size_t)stride16 * 16 * mb);   // (by way of an integer it would no longer count as global memory)
}
template <typename TX, typename T, typename TO, int NCH, int RW>
__global__ __launch_bounds__(kLnThreads) void ln_fwd_kernel(
    const TX* __restrict__ x0, const T* __restrict__ gamma, const T* __restrict__ beta, TO* __restrict__ out0,
    float* __restrict__ mean0, float* __restrict__ rstd0, float* __restrict__ xcopy0, int T_rows, int H, float eps,
    uint32_t stride16, uint32_t x_stride16) {
  const TX* __restrict__ x = at_mb(x0, x_stride16, blockIdx.y);
  TO* __restrict__ out = at_mb(out0, stride16, blockIdx.y);
  float* __restrict__ mean = at_mb(mean0, stride16, blockIdx.y);
  float* __restrict__ rstd = at_mb(rstd0, stride16, blockIdx.y);
  float* __restrict__ xcopy = xcopy0 ? at_mb(xcopy0, stride16, blockIdx.y) : nullptr;
  constexpr int NWV = kLnThreads / kWave, NT = RW * kWave;   // NT: threads of a row
  static_assert(RW == 1 || RW == NWV, "a wave or the workgroup per row");
  __shared__ float red[2][NWV];
  const int t = threadIdx.x % NT;
  const int row = blockIdx.x * (NWV / RW) + threadIdx.x / NT;
  if (RW == 1 && row >= T_rows) return;
  const int nvec = H / 8;
  const TX* xr = x + (size_t)row * H;
  float xv[NCH][8];
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int i = t + c * NT;
    if (i < nvec) load8(xr + (size_t)i * 8, xv[c]);
  }
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int i = t + c * NT;
    if (i < nvec) {
      if (xcopy) store8(xcopy + (size_t)row * H + (size_t)i * 8, xv[c]);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += xv[c][e];
    }
  }
  const float mu = block_sum<RW>(s, red[0]) / (float)H;
  float q = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int i = t + c * NT;
    if (i < nvec) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float d = xv[c][e] - mu;
        q += d * d;
      }
    }
  }
  const float var = block_sum<RW>(q, red[1]) / (float)H;
  const float r = 1.f / sqrtf(var + eps);
  TO* orow = out + (size_t)row * H;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int i = t + c * NT;
    if (i < nvec) {
      float g[8], b[8], o[8];
      load8(gamma + (size_t)i * 8, g);
      load8(beta + (size_t)i * 8, b);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (xv[c][e] - mu) * r * g[e] + b[e];
      store8(orow + (size_t)i * 8, o);
    }
  }
  if (t == 0) {
    mean[row] = mu;
    rstd[row] = r;
  }
}

// For every matrix: partial[slice][n] = sum over the slice's rows (4 slice + w, then every 4 slices) of A[m][n].
// Lane owns one 16-byte column vector; four waves (w) take interleaved rows and are combined through their LDS `sm`
// in fixed order.  One launch takes all the matrices of a layer (the same M rows): below some MB each is a few
// microseconds of launch and latency whatever its size.  Three matrices of 128 rows, 128 to 512 columns, in one
// launch instead of three: 3.7 us of a 74 us step.
// NM: matrices there is room for; one alone has a form of its own, without the search.
template <int NM> struct ColsumArgs {
  ColsumMat mat[NM];
  int first[NM];   // first x of a matrix
  uint32_t stride16;
};
template <typename T, int NM>
__device__ __forceinline__ void colsum_partial(const ColsumArgs<NM>& args, int M, int x, int slice, int slices, int mb, int w,
                                               float* sm) {
  constexpr int V = Vec16<T>::N;
  int k = 0;
#pragma unroll
  for (int i = 1; i < NM; ++i)
    if (x >= args.first[i]) k = i;
  const int N = args.mat[k].N;
  const T* __restrict__ A = at_mb(static_cast<const T*>(args.mat[k].A), args.stride16, mb);
  float* __restrict__ partial = args.mat[k].partial + (size_t)mb * slices * N;
  const int lane = threadIdx.x & (kWave - 1);
  const int col = ((x - args.first[k]) * kWave + lane) * V;
  float acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = 0.f;
  if (col < N) {
    for (int m = slice * 4 + w; m < M; m += slices * 4) {
      const Vec16<T> v = load16(A + (size_t)m * N + col);
#pragma unroll
      for (int e = 0; e < V; ++e) acc[e] += v.get(e);
    }
  }
#pragma unroll
  for (int e = 0; e < V; ++e) sm[w * kWave * V + lane * V + e] = acc[e];
  __syncthreads();
  if (w == 0 && col < N && slice < slices) {
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const int i = lane * V + e;
      partial[(size_t)slice * N + col + e] = sm[i] + sm[kWave * V + i] + sm[2 * kWave * V + i] + sm[3 * kWave * V + i];
    }
  }
}

// ----------------------------------------------------------------- LN bwd ----
// Per token, with xhat = (x-mu) r and g = dout*gamma:
//   dx = dres + r (g - mean(g) - xhat mean(g xhat)).
// A workgroup's 8 waves form 8/RW groups of RW waves, a row per group at a time; each group keeps its
// share of sum_t dout*xhat and sum_t dout in registers, the groups add up through LDS in fixed order
// at the end, and the workgroup writes partial[blockIdx.x][0][H] / [1][H] for the reduction below.
// With DXSUM it also keeps the column sums of dx as stored (partial[blockIdx.x][2][H]): dx is the
// gradient of the output of the linear layer in front of the residual branch, so these
// are that layer's bias gradient, which then needs no pass of its own over dx.
// Bound by HBM, and by the partial sums where rows are short.  A wave per row up to 1024 columns (no
// barrier, no idle threads, an eighth of the partial sums): 4096 rows of 1024 with the reduction
// 23.1 -> 12.8 us, 8192 of 512 30.4 -> 11.7 us; 3968 of 2048 26.6 -> 20.7 us; 16-bit operands kept
// packed and rows up to 12288 in three chunks, prefetched: 2048 of 12288 95.5 -> 65.3 us (3.9 TB/s).
constexpr int kLnBwdThreads = 512;
// Workgroups: 512 for rows of a whole workgroup (measured at 4096 rows of 4096: 256 -> 42.6 us,
// 512 -> 39.6, 1024 -> 50.2: more workgroups put more rows in flight but each writes its own partial
// sums), 256 where a workgroup has several rows in flight.
constexpr int kLnBwdMaxBlocks = 512, kLnBwdMaxBlocksGroups = 256;
int ln_bwd_row_waves(int H) { return H <= 1024 ? 1 : (H <= 2048 ? 4 : 8); }
int ln_bwd_blocks(int T_rows, int H) {
  const int groups = kLnBwdThreads / kWave / ln_bwd_row_waves(H), most = groups == 1 ? kLnBwdMaxBlocks : kLnBwdMaxBlocksGroups;
  const int need = (T_rows + groups - 1) / groups;
  return need < most ? need : most;
}

// NM > 0: the workgroups from `tail.blocks` on take the column sums of up to NM matrices of the same rows, two slices
// each (see ln_bwd_takes_colsums()).
template <int NM> struct LnBwdTail {
  ColsumArgs<NM> cols;
  int blocks, nx, slices;   // workgroups of the LayerNorm; x and slices of the column sums
};
template <> struct LnBwdTail<0> {};
template <typename TX, typename T, int NCH, int RW, bool DXSUM, int NM>
__global__ __launch_bounds__(kLnBwdThreads) void ln_bwd_kernel(
    const T* __restrict__ dout0, const TX* __restrict__ x0, const float* __restrict__ mean0,
    const float* __restrict__ rstd0, const T* __restrict__ gamma, const T* __restrict__ dres0,
    T* __restrict__ dx0, float* __restrict__ partial0, int T_rows, int H, uint32_t act16, uint32_t dres16, uint32_t dx16,
    const LnBwdTail<NM> tail) {
  constexpr int NWV = kLnBwdThreads / kWave, GR = NWV / RW, NT = RW * kWave, NPART = DXSUM ? 3 : 2;
  constexpr int COMB = GR > 1 ? GR * NT * NCH * 8 : 4, SUMS = NM > 0 ? NWV * kWave * Vec16<T>::N : 4;
  __shared__ __attribute__((aligned(16))) float comb[COMB > SUMS ? COMB : SUMS];
  int n_blocks = gridDim.x;
  if constexpr (NM > 0) {
    n_blocks = tail.blocks;
    if ((int)blockIdx.x >= n_blocks) {
      const int r = blockIdx.x - n_blocks, half = threadIdx.x / (4 * kWave);   // (four waves a slice)
      colsum_partial<T>(tail.cols, T_rows, r % tail.nx, r / tail.nx * 2 + half, tail.slices, blockIdx.y, threadIdx.x / kWave % 4,
                        comb + half * (4 * kWave * Vec16<T>::N));
      return;
    }
  }
  const T* __restrict__ dout = at_mb(dout0, act16, blockIdx.y);
  const TX* __restrict__ x = at_mb(x0, act16, blockIdx.y);
  const float* __restrict__ mean = at_mb(mean0, act16, blockIdx.y);
  const float* __restrict__ rstd = at_mb(rstd0, act16, blockIdx.y);
  const T* __restrict__ dres = dres0 ? at_mb(dres0, dres16, blockIdx.y) : nullptr;
  T* __restrict__ dx = at_mb(dx0, dx16, blockIdx.y);
  float* __restrict__ partial = partial0 + (size_t)blockIdx.y * n_blocks * (DXSUM ? 3 : 2) * H;
  // At most one barrier per row: the two row sums are reduced together and the LDS slots alternate
  // between rows, so a row's writes cannot overtake the previous row's reads.  The loads of
  // the next row (when the row fits few registers) and of the residual gradient are issued
  // before the barrier, so that memory latency overlaps the reduction.
  constexpr bool PREFETCH = NCH <= 3;   // 168 registers at three chunks; a fourth would spill
  __shared__ float red[2][2][NWV];
  const int nvec = H / 8;
  const int wv = threadIdx.x / kWave, grp = wv / RW, t = threadIdx.x % NT;
  float dg[NCH][8], db[NCH][8], dc[DXSUM ? NCH : 1][8];
  Raw8<T> gam[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int i = t + c * NT;
    if (i < nvec) gam[c].load(gamma + (size_t)i * 8);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      dg[c][e] = db[c][e] = 0.f;
      if constexpr (DXSUM) dc[c][e] = 0.f;
    }
  }
  Raw8<T> dv[NCH], dvn[PREFETCH ? NCH : 1];
  float xh[NCH][8], xn[PREFETCH ? NCH : 1][8];
  auto load_row = [&](int row, Raw8<T>(&d)[NCH], float (&xx)[NCH][8]) {
    const size_t base = (size_t)row * H;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int i = t + c * NT;
      if (i < nvec) {
        d[c].load(dout + base + (size_t)i * 8);
        load8(x + base + (size_t)i * 8, xx[c]);
      }
    }
  };
  const int step = n_blocks * GR;
  if constexpr (PREFETCH) {
    if ((int)blockIdx.x * GR + grp < T_rows) load_row(blockIdx.x * GR + grp, dv, xh);
  }
  int buf = 0;
  for (int first = blockIdx.x * GR; first < T_rows; first += step, buf ^= 1) {
    const int row = first + grp;
    const bool on = GR == 1 || row < T_rows;      // the groups of a workgroup meet at the barriers together
    if constexpr (!PREFETCH) {
      if (on) load_row(row, dv, xh);
    }
    const float mu = on ? mean[row] : 0.f, r = on ? rstd[row] : 0.f;
    const size_t base = (size_t)row * H;
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int i = t + c * NT;
      if (on && i < nvec) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float d = dv[c].get(e);
          xh[c][e] = (xh[c][e] - mu) * r;
          const float g = d * gam[c].get(e);
          s1 += g;
          s2 += g * xh[c][e];
          dg[c][e] += d * xh[c][e];
          db[c][e] += d;
        }
      }
    }
    if constexpr (NCH == 4) {
      // form dout * gamma anew below: kept across the reduction it spilled 29 registers (2048 rows of 16384
      // with the sums of dx 144 -> 109 us, 8192 of 12800 374 -> 231)
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        dv[c].opaque();
        gam[c].opaque();
      }
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (RW > 1 && (threadIdx.x & (kWave - 1)) == 0) {
      red[buf][0][wv] = s1;
      red[buf][1][wv] = s2;
    }
    Raw8<T> rs[NCH];
    if (dres) {
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int i = t + c * NT;
        if (on && i < nvec) rs[c].load(dres + base + (size_t)i * 8);
      }
    }
    if constexpr (PREFETCH) {
      const int nxt = row + step;
      if (nxt < T_rows) load_row(nxt, dvn, xn);
    }
    float m1 = s1, m2 = s2;
    if constexpr (RW > 1) {
      __syncthreads();
      m1 = m2 = 0.f;
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        m1 += red[buf][0][grp * RW + i];
        m2 += red[buf][1][grp * RW + i];
      }
    }
    m1 /= (float)H;
    m2 /= (float)H;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int i = t + c * NT;
      if (on && i < nvec) {
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float v = r * (dv[c].get(e) * gam[c].get(e) - m1 - xh[c][e] * m2);
          if (dres) v += rs[c].get(e);
          o[e] = v;
          if constexpr (DXSUM) dc[c][e] += (float)(T)v;
        }
        store8(dx + base + (size_t)i * 8, o);
      }
    }
    if constexpr (PREFETCH) {
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        dv[c] = dvn[c];
#pragma unroll
        for (int e = 0; e < 8; ++e) xh[c][e] = xn[c][e];
      }
    }
  }
  float* pg = partial + (size_t)blockIdx.x * NPART * H;
  auto write_part = [&](float (&v)[NCH][8], int part) {
    if constexpr (GR == 1) {
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int i = t + c * NT;
        if (i < nvec) store8(pg + (size_t)part * H + (size_t)i * 8, v[c]);
      }
    } else {
      constexpr int PITCH = NT * NCH * 8;   // floats of a group's sums
      __syncthreads();
#pragma unroll
      for (int c = 0; c < NCH; ++c) store8(comb + grp * PITCH + (t + c * NT) * 8, v[c]);
      __syncthreads();
      for (int i = threadIdx.x * 4; i < H; i += kLnBwdThreads * 4) {
        f32x4 a = *reinterpret_cast<const f32x4*>(comb + i);
#pragma unroll
        for (int k = 1; k < GR; ++k) a += *reinterpret_cast<const f32x4*>(comb + k * PITCH + i);
        *reinterpret_cast<f32x4*>(pg + (size_t)part * H + i) = a;
      }
    }
  };
  write_part(dg, 0);
  write_part(db, 1);
  if constexpr (DXSUM) write_part(dc, 2);
}

template <int NS, int NB> __global__ __launch_bounds__(256) void reduce_partials_kernel(const ReduceArgs<NS> args) {
  __shared__ float sm[NB][32][33];
  reduce_columns<NS, NB>(args, blockIdx.x, sm);
}

template <int NS, int NB> static hipError_t launch_reduce(const ReduceSeg* segs, int n, hipStream_t st) {
  ReduceArgs<NS> a{};
  const int blocks = reduce_layout<NS>(segs, n, &a);
  hipLaunchKernelGGL((reduce_partials_kernel<NS, NB>), dim3(blocks), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t reduce_partials(const ReduceSeg* segs, int n, hipStream_t st) {
  if (n < 1 || n > kMaxReduceSegs) return hipErrorInvalidValue;
  bool window = false;
  for (int i = 0; i < n; ++i) {
    if (segs[i].batch < 1 || segs[i].batch > kMaxWindow) return hipErrorInvalidValue;
    window = window || segs[i].batch > 1;
  }
  if (window) return n == 1 ? launch_reduce<1, kMaxWindow>(segs, n, st) : launch_reduce<kMaxReduceSegs, kMaxWindow>(segs, n, st);
  return n == 1 ? launch_reduce<1, 1>(segs, n, st) : launch_reduce<kMaxReduceSegs, 1>(segs, n, st);
}

// ----------------------------------------------------------------- colsum ----
// In a launch of its own; blockIdx.z: the micro-batch.
template <typename T, int NM>
__global__ __launch_bounds__(256) void colsum_partial_kernel(const ColsumArgs<NM> args, int M) {
  __shared__ float sm[4 * kWave * Vec16<T>::N];
  colsum_partial<T>(args, M, blockIdx.x, blockIdx.y, gridDim.y, blockIdx.z, threadIdx.x / kWave, sm);
}

// --------------------------------------------------------------- launchers ----
template <typename TX, typename T, typename TO>
static hipError_t ln_fwd_t(int T_rows, int H, float eps, const void* x, const void* gamma, const void* beta,
                           void* out, float* mean, float* rstd, float* xcopy, hipStream_t st, int n, size_t stride,
                           size_t x_stride) {
  if (n < 1 || n > kMaxWindow || !window_stride_ok(stride) || !window_stride_ok(x_stride)) return hipErrorInvalidValue;
#define GPTS_LN_FWD(N, RW)                                                                                        \
  hipLaunchKernelGGL((ln_fwd_kernel<TX, T, TO, N, RW>), dim3(RW == 1 ? (T_rows + 3) / 4 : T_rows, n), dim3(kLnThreads), 0, st, \
                     (const TX*)x, (const T*)gamma, (const T*)beta, (TO*)out, mean, rstd, xcopy, T_rows, H, eps,    \
                     (uint32_t)(stride / 16), (uint32_t)(x_stride / 16))
  // A wave per row up to 2048 columns (32 registers a lane), a workgroup beyond -- and for many long rows
  // too, where a wave's four chunks each wait for memory longer than the barrier costs.  Workgroup | wave,
  // us: fp32 4096x2048 15.1 | 13.8, 8192x1536 17.4 | 19.1, 16384x2048 42.9 | 46.0, 32768x2048 100 | 113,
  // 32768x1152 67.1 | 65.0; fp32 in, 16 bits out 16384x2048 31.2 | 30.7, 32768x1792 60.9 | 61.4, 32768x2048
  // 69.1 | 72.1; 16 bits in and out 65536x2048 105 | 96.
  const bool wave_row = H <= 1152 || sizeof(TX) == 2 ||
                        (sizeof(TO) == 4 ? T_rows <= 4096 : (H <= 1792 || T_rows <= 16384));
  if (H <= 512) GPTS_LN_FWD(1, 1);
  else if (H <= 1024) GPTS_LN_FWD(2, 1);
  else if (H <= 2048 && wave_row) GPTS_LN_FWD(4, 1);
  else if (H <= 2048) GPTS_LN_FWD(1, 4);
  else if (H <= 4096) GPTS_LN_FWD(2, 4);
  else if (H <= 8192) GPTS_LN_FWD(4, 4);
  else GPTS_LN_FWD(8, 4);
#undef GPTS_LN_FWD
  return hipGetLastError();
}

hipError_t ln_fwd(int dtype, bool x_f32, int T_rows, int H, float eps, const void* x,
                  const void* gamma, const void* beta, void* out, float* mean, float* rstd,
                  hipStream_t st, bool out_f16, float* xcopy, int n, size_t stride, size_t x_stride) {
#define GPTS_LN(TX, T, TO) ln_fwd_t<TX, T, TO>(T_rows, H, eps, x, gamma, beta, out, mean, rstd, xcopy, st, n, stride, x_stride)
  if (dtype == 0) return out_f16 ? hipErrorInvalidValue : GPTS_LN(float, float, float);
  if (x_f32) return out_f16 ? GPTS_LN(float, bf16, f16) : GPTS_LN(float, bf16, bf16);
  return out_f16 ? GPTS_LN(bf16, bf16, f16) : GPTS_LN(bf16, bf16, bf16);
#undef GPTS_LN
}

static int colsum_splits(int M) { return M < 4 * 64 ? (M + 3) / 4 : 64; }
// the matrices' places in a launch and the sums they leave; returns how many x there are
template <int NM>
static int colsum_layout(int dtype, int M, const ColsumMat* mats, int n, ReduceSeg* segs, int batch, size_t stride, ColsumArgs<NM>* a) {
  const int V = dtype == 0 ? 4 : 8;
  int blocks = 0;
  for (int i = 0; i < NM; ++i) {
    a->first[i] = i < n ? blocks : 0x7fffffff;      // (never reached)
    if (i >= n) continue;
    a->mat[i] = mats[i];
    blocks += (mats[i].N / V + kWave - 1) / kWave;
    segs[i] = colsum_segment(mats[i].partial, colsum_splits(M), mats[i].N, mats[i].out);
    segs[i].batch = batch;
  }
  a->stride16 = (uint32_t)(stride / 16);
  return blocks;
}

template <typename TX, typename T, int NM>
static hipError_t ln_bwd_t(int T_rows, int H, const void* dout, const void* x, const float* mean,
                           const float* rstd, const void* gamma, const void* dres, void* dx, bool dxsum,
                           float* partial, const LnBwdWindow& win, const LnBwdTail<NM>& tail, int tail_blocks, hipStream_t st) {
  const dim3 g(ln_bwd_blocks(T_rows, H) + tail_blocks, win.n), b(kLnBwdThreads);
#define GPTS_LN_BWD_(N, RW, SUM)                                                                                  \
  hipLaunchKernelGGL((ln_bwd_kernel<TX, T, N, RW, SUM, NM>), g, b, 0, st, (const T*)dout, (const TX*)x, mean, rstd,   \
                     (const T*)gamma, (const T*)dres, (T*)dx, partial, T_rows, H, (uint32_t)(win.act / 16),         \
                     (uint32_t)(win.dres / 16), (uint32_t)(win.dx / 16), tail)
#define GPTS_LN_BWD(N, RW)                  \
  do {                                      \
    if (dxsum) GPTS_LN_BWD_(N, RW, true);   \
    else GPTS_LN_BWD_(N, RW, false);        \
  } while (0)
  if (H <= 512) GPTS_LN_BWD(1, 1);
  else if (H <= 1024) GPTS_LN_BWD(2, 1);
  else if (H <= 2048) GPTS_LN_BWD(1, 4);
  else if constexpr (NM > 0) return hipErrorInvalidValue;
  else if (H <= 4096) GPTS_LN_BWD(1, 8);
  else if (H <= 8192) GPTS_LN_BWD(2, 8);
  else if (H <= 12288) GPTS_LN_BWD(3, 8);
  else GPTS_LN_BWD(4, 8);
#undef GPTS_LN_BWD
#undef GPTS_LN_BWD_
  return hipGetLastError();
}

// Whether the column sums go into the LayerNorm's launch.  Small ones are a launch that leaves most of the chip idle,
// and run beside it; large ones fill it alone in smaller workgroups, of which a unit holds more than of those with
// the LayerNorm's registers, and long rows leave a unit one workgroup.  Apart | together, us, bf16, rows x hidden and
// the matrices' columns: 384x320 and 960 7.6 | 4.9; 2048x2048 and 6144 19.9 | 15.7, 8192 22.1 | 20.0; 4096x1024 and
// 3072 20.4 | 18.7, 4096 20.9 | 20.6; 2048x5120 and 15360 41 | 50, 20480 49 | 61; 2048x12288 and 4608 74 | 72, 16896
// 84 | 92.
bool ln_bwd_takes_colsums(int dtype, int T_rows, int H, const ColsumMat* cols, int n) {
  size_t bytes = 0;
  for (int i = 0; i < n; ++i) bytes += (size_t)T_rows * cols[i].N * (dtype == 0 ? 4 : 2);
  return H <= 2048 && bytes <= (size_t)32 << 20;
}
template <int NM>
static hipError_t ln_bwd_any(int dtype, bool x_f32, int T_rows, int H, const void* dout, const void* x, const float* mean,
                             const float* rstd, const void* gamma, const void* dres, void* dx, bool dxsum, float* partial,
                             const LnBwdWindow& w, const LnBwdTail<NM>& tail, int tail_blocks, hipStream_t st) {
#define GPTS_LN_BWD(TX, T) ln_bwd_t<TX, T, NM>(T_rows, H, dout, x, mean, rstd, gamma, dres, dx, dxsum, partial, w, tail, tail_blocks, st)
  if (dtype == 0) return GPTS_LN_BWD(float, float);
  return x_f32 ? GPTS_LN_BWD(float, bf16) : GPTS_LN_BWD(bf16, bf16);
#undef GPTS_LN_BWD
}
hipError_t ln_bwd_partials(int dtype, bool x_f32, int T_rows, int H, const void* dout, const void* x,
                           const float* mean, const float* rstd, const void* gamma, const void* dres, void* dx,
                           float* dgamma, float* dbeta, float* dxsum, float* partial, ReduceSeg* seg, hipStream_t st,
                           const LnBwdWindow* win, const ColsumMat* cols, int n_cols, ReduceSeg* col_segs) {
  if (H > 4 * 8 * kLnBwdThreads || (win && (win->n < 1 || win->n > kMaxWindow))) return hipErrorInvalidValue;
  if (n_cols < 0 || n_cols > kMaxColsums) return hipErrorInvalidValue;
  const int np = dxsum ? 3 : 2;
  const LnBwdWindow w = win ? *win : LnBwdWindow();
  if (!window_stride_ok(w.act) || !window_stride_ok(w.dres) || !window_stride_ok(w.dx) || !window_stride_ok(w.cols)) return hipErrorInvalidValue;
  const int blocks = ln_bwd_blocks(T_rows, H);
  *seg = ReduceSeg{partial, (size_t)np * H, blocks, np * H, H, 2 * H, dgamma, dbeta, dxsum, w.n};
  if (!n_cols)
    return ln_bwd_any<0>(dtype, x_f32, T_rows, H, dout, x, mean, rstd, gamma, dres, dx, dxsum, partial, w, LnBwdTail<0>(), 0, st);
  LnBwdTail<kMaxColsums> tail{};
  tail.nx = colsum_layout(dtype, T_rows, cols, n_cols, col_segs, w.n, w.cols, &tail.cols);
  tail.blocks = blocks;
  tail.slices = colsum_splits(T_rows);
  return ln_bwd_any<kMaxColsums>(dtype, x_f32, T_rows, H, dout, x, mean, rstd, gamma, dres, dx, dxsum, partial, w, tail,
                                 tail.nx * ((tail.slices + 1) / 2), st);
}
hipError_t ln_bwd(int dtype, bool x_f32, int T_rows, int H, const void* dout, const void* x,
                  const float* mean, const float* rstd, const void* gamma, const void* dres, void* dx,
                  float* dgamma, float* dbeta, float* dxsum, float* partial, hipStream_t st) {
  ReduceSeg seg;
  const hipError_t e = ln_bwd_partials(dtype, x_f32, T_rows, H, dout, x, mean, rstd, gamma, dres, dx, dgamma, dbeta, dxsum,
                                       partial, &seg, st);
  return e != hipSuccess ? e : reduce_partials(&seg, 1, st);
}

// g[i] = gelu(u[i]), 8 elements per thread (recomputation of the MLP activation)
template <typename TU, typename T, int KIND>
__global__ __launch_bounds__(256) void gelu_kernel(const TU* __restrict__ u, T* __restrict__ g, size_t n8) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n8) return;
  float v[8];
  load8(u + i * 8, v);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = gelu_f<KIND>(v[e]);
  store8(g + i * 8, v);
}

hipError_t gelu_fwd(int dtype, int kind, const void* u, void* g, size_t n, hipStream_t st, bool u_f16) {
  const size_t n8 = n / 8;
  dim3 grid((unsigned)((n8 + 255) / 256)), blk(256);
  if (dtype == 0) {
    if (u_f16) return hipErrorInvalidValue;
    if (kind == 0) hipLaunchKernelGGL((gelu_kernel<float, float, 0>), grid, blk, 0, st, (const float*)u, (float*)g, n8);
    else hipLaunchKernelGGL((gelu_kernel<float, float, 1>), grid, blk, 0, st, (const float*)u, (float*)g, n8);
  } else if (u_f16) {
    if (kind == 0) hipLaunchKernelGGL((gelu_kernel<f16, bf16, 0>), grid, blk, 0, st, (const f16*)u, (bf16*)g, n8);
    else hipLaunchKernelGGL((gelu_kernel<f16, bf16, 1>), grid, blk, 0, st, (const f16*)u, (bf16*)g, n8);
  } else {
    if (kind == 0) hipLaunchKernelGGL((gelu_kernel<bf16, bf16, 0>), grid, blk, 0, st, (const bf16*)u, (bf16*)g, n8);
    else hipLaunchKernelGGL((gelu_kernel<bf16, bf16, 1>), grid, blk, 0, st, (const bf16*)u, (bf16*)g, n8);
  }
  return hipGetLastError();
}

// out[i] = bf16(in[i]) for fp16 in: the backward phase's bf16 copies of forward activations
// that were stored in fp16
__global__ __launch_bounds__(256) void f16_to_bf16_kernel(const f16* __restrict__ in, bf16* __restrict__ out,
                                                          size_t n8) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n8) return;
  float v[8];
  load8(in + i * 8, v);
  store8(out + i * 8, v);
}
hipError_t f16_to_bf16(const void* in, void* out, size_t n, hipStream_t st) {
  const size_t n8 = n / 8;
  hipLaunchKernelGGL(f16_to_bf16_kernel, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, st, (const f16*)in,
                     (bf16*)out, n8);
  return hipGetLastError();
}

size_t ln_bwd_scratch_bytes(int T_rows, int H) {
  return (size_t)ln_bwd_blocks(T_rows, H) * 3 * H * sizeof(float);
}

size_t colsum_scratch_bytes(int M, int N) { return (size_t)colsum_splits(M) * N * sizeof(float); }

ReduceSeg colsum_segment(const float* partial, int G, int N, float* out) {
  return ReduceSeg{partial, (size_t)N, G, N, N, N, out, nullptr, nullptr, 1};
}
template <int NM>
static hipError_t launch_colsum(int dtype, int M, const ColsumMat* mats, int n, ReduceSeg* segs, hipStream_t st, int batch,
                                size_t stride) {
  ColsumArgs<NM> a{};
  const int blocks = colsum_layout(dtype, M, mats, n, segs, batch, stride, &a);
  const dim3 g(blocks, colsum_splits(M), batch);
  if (dtype == 0) hipLaunchKernelGGL((colsum_partial_kernel<float, NM>), g, dim3(256), 0, st, a, M);
  else hipLaunchKernelGGL((colsum_partial_kernel<bf16, NM>), g, dim3(256), 0, st, a, M);
  return hipGetLastError();
}
hipError_t colsum_partials(int dtype, int M, const ColsumMat* mats, int n, ReduceSeg* segs, hipStream_t st, int batch,
                           size_t stride) {
  if (n < 1 || n > kMaxColsums || batch < 1 || !window_stride_ok(stride)) return hipErrorInvalidValue;
  return n == 1 ? launch_colsum<1>(dtype, M, mats, n, segs, st, batch, stride)
                : launch_colsum<kMaxColsums>(dtype, M, mats, n, segs, st, batch, stride);
}

struct CopyTable {
  const void* src[kMaxWindow];
  void* dst[kMaxWindow];
};
__global__ __launch_bounds__(256) void window_copy_kernel(const CopyTable t, size_t n16) {
  const f32x4* const s = static_cast<const f32x4*>(t.src[blockIdx.y]);
  f32x4* const d = static_cast<f32x4*>(t.dst[blockIdx.y]);
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) d[i] = s[i];
}
hipError_t window_copy(int n, const void* const* src, void* const* dst, size_t bytes, hipStream_t st) {
  if (n < 1 || n > kMaxWindow || bytes % 16) return hipErrorInvalidValue;
  CopyTable t;
  for (int m = 0; m < kMaxWindow; ++m) {
    t.src[m] = src[m < n ? m : 0];
    t.dst[m] = dst[m < n ? m : 0];
  }
  const size_t n16 = bytes / 16, blocks = (n16 + 1023) / 1024;   // up to four vectors a thread, then more
  hipLaunchKernelGGL(window_copy_kernel, dim3((unsigned)(blocks < 2048 ? blocks : 2048), n), dim3(256), 0, st, t, n16);
  return hipGetLastError();
}
hipError_t colsum(int dtype, int M, int N, const void* A, float* out, float* partial, hipStream_t st) {
  const ColsumMat mat{A, N, out, partial};
  ReduceSeg seg;
  const hipError_t e = colsum_partials(dtype, M, &mat, 1, &seg, st);
  return e != hipSuccess ? e : reduce_partials(&seg, 1, st);
}

// ---- column sums for callers that cannot allocate ------------------------------------------
// gpt_stage_op_colsum needs a scratch buffer for its per-workgroup partial sums.  This variant
// takes them from a fixed array in device memory instead, so the call allocates nothing: for
// callers under HIP graph capture, in tight serving loops, or in harnesses that forbid
// hipMalloc.  Each GPU the library runs on holds its own copy of the array (4 MiB) until the
// process ends.  In host code the array's name is only a stand-in: its device address is looked
// up once per device and that pointer is what the kernels get.
namespace {
constexpr int kNoAllocMaxN = 16384;   // columns; colsum_splits() never exceeds 64 rows of partials
constexpr int kNoAllocMaxDevices = 64;
static __device__ __align__(256) float scratch[64 * kNoAllocMaxN];
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kNoAllocMaxDevices] = {};

// device address of `scratch` on the current device (looked up on first use per device)
hipError_t scratch_on_current_device(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kNoAllocMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}
}  // namespace
}  // namespace gpts

extern "C" int gpt_stage_op_colsum_noalloc(int dtype, int M, int N, const void* A, float* colsum_out,
                                           void* stream) {
  using namespace gpts;
  if ((dtype != GPTS_FP32 && dtype != GPTS_BF16) || !A || !colsum_out)
    return set_error(GPTS_EINVAL, "colsum_noalloc: bad argument");
  if (M < 1 || N < 8 || N % 8) return set_error(GPTS_ESHAPE, "colsum_noalloc: N must be a multiple of 8");
  if (N > kNoAllocMaxN || colsum_scratch_bytes(M, N) > sizeof(float) * 64 * (size_t)kNoAllocMaxN)
    return set_error(GPTS_ESHAPE, "colsum_noalloc: N exceeds 16384, the size the built-in scratch array is made for");
  float* partial = nullptr;
  hipError_t e = scratch_on_current_device(&partial);
  if (e == hipSuccess) e = colsum(dtype, M, N, A, colsum_out, partial, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return set_error(GPTS_EHIP, hipGetErrorString(e));
  return GPTS_OK;
}

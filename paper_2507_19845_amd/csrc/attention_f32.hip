// Causal softmax attention of fp32 stages on the matrix cores (v_mfma_f32_16x16x4_f32: fp32
// multiply-add and accumulation), for 16-byte aligned buffers; attention_simple.hip takes the rest.
//
// A workgroup owns 16 rows (queries in the forward pass and for dQ, keys for dK and dV) and its four
// waves share out the 16-row blocks of the other side: block w, w+4, ... to wave w.  Every block is
// read by one wave of the workgroup only, so operands go straight from memory (the L2, mostly) to
// registers.  The waves' partial results meet in LDS at the end and are added in fixed order.
// All products are computed transposed, so that an accumulator is, register by register, the B
// operand of the next product: lane l owns column l%16 (its query or key), and accumulator register
// r holds row 4*(l/16) + r.
//   forward   S^T = K Q^T,  O^T += V^T P^T                                     (online softmax)
//   dQ        S^T = K Q^T,  dP^T = V dO^T,  dQ^T += K^T dS^T
//   dK, dV    S = Q K^T,    dP = dO V^T,    dV^T += dO^T P,  dK^T += Q^T dS
// with P = exp(S/sqrt(D) - lse), dS = P (dP - delta) / sqrt(D), delta = rowsum(dO o O).  dQ and
// dK/dV are two kinds of workgroup of ONE launch: each forms the delta it needs itself.
//
// Only the block on the diagonal has masked entries.  Their probabilities are 0, but 0 times an
// infinity or a NaN in the masked row would still enter the product, so that block's right-hand rows
// are checked and, if any is not finite, its product is formed element by element.
//
// Bound: latency and the fp32 matrix pipe; 16 rows per workgroup because fp32 stages are small
// (B=2, 4 heads of 32, S=64: 32 workgroups where 64-row ones would be 8).  Measured against the FMA
// kernels of attention_simple.hip, forward / backward: B=2 S=64, 4 heads of 32: 46 -> 3.8 / 90 -> 5.2 us;
// B=3 S=333, 8 heads of 64: 230 -> 13.7 / 522 -> 46 us.
#include <type_traits>

#include "kernels.hpp"

namespace gpts {
namespace {

constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
// stands for "no key seen yet" in the running maximum: no finite logit is smaller, and the
// difference of two such values is 0 and not NaN
constexpr float kNoKey = -3.4028234663852886e38f;

// Row fragment: row `row` (one per lane%16), elements 16q + 4*(lane/16) .. +3 in v[q].  Rows past the
// end read as zero.
template <int D> struct RowFrag {
  f32x4 v[D / 16];
  __device__ __forceinline__ void load(const float* X, size_t ld, int row, int S, int g) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const float* p = X + (size_t)(row < S ? row : 0) * ld + 4 * g;
#pragma unroll
    for (int q = 0; q < D / 16; ++q) v[q] = row < S ? *reinterpret_cast<const f32x4*>(p + 16 * q) : zero;
  }
};
// The block index db and row-in-block rho of a transposed accumulator stand for element
//   d = (db / VW) * 16*VW + VW*rho + db % VW
// (VW blocks interleaved), so that a lane reads VW blocks' elements of one row at once.
template <int D> struct ColMap {
  static constexpr int VW = D == 32 ? 2 : 4, NG = D / 16 / VW;
  static __device__ __forceinline__ int d_of(int group, int rho) { return group * 16 * VW + VW * rho; }
};
// Column fragment of rows row0 + 4*(lane/16) + r: element rho = lane%16 of every block.
template <int D> struct ColFrag {
  float v[4][D / 16];
  __device__ __forceinline__ void load(const float* X, size_t ld, int row0, int S, int g, int i) {
    using M = ColMap<D>;
    typedef float vec __attribute__((ext_vector_type(M::VW)));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row0 + 4 * g + r;
      const float* p = X + (size_t)(row < S ? row : 0) * ld;
#pragma unroll
      for (int gr = 0; gr < M::NG; ++gr) {
        const vec x = *reinterpret_cast<const vec*>(p + M::d_of(gr, i));
#pragma unroll
        for (int e = 0; e < M::VW; ++e) v[r][gr * M::VW + e] = row < S ? x[e] : 0.f;
      }
    }
  }
  __device__ __forceinline__ bool finite() const {
    float z = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int db = 0; db < D / 16; ++db) z = fmaf(v[r][db], 0.f, z);
    return z == 0.f;
  }
};

// S (or dP) block: rows of `a` against columns of `b`
template <int D> __device__ __forceinline__ f32x4 rows_times_cols(const RowFrag<D>& a, const RowFrag<D>& b) {
  f32x4 s[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};   // two chains: half the dependent latency
#pragma unroll
  for (int q = 0; q < D / 16; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) s[q & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[q][e], b.v[q][e], s[q & 1], 0, 0, 0);
  return s[0] + s[1];
}
// acc^T[d][col] += sum over the block's 16 rows of X[row][d] * w[row][col]
template <int D> __device__ __forceinline__ void accumulate(f32x4 (&acc)[D / 16], const ColFrag<D>& x, const f32x4& w) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int db = 0; db < D / 16; ++db) acc[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[r][db], w[r], acc[db], 0, 0, 0);
}
// The same for the diagonal block, whose entries with !allowed(row, column) do not count (w is 0
// there): exact also when X holds values that are not finite.
template <int D, class Allowed>
__device__ __forceinline__ void accumulate_diagonal(f32x4 (&acc)[D / 16], const ColFrag<D>& x, const f32x4& w, const float* X,
                                                    size_t ld, int row0, int S, int g, int i, Allowed&& allowed) {
  if (__builtin_amdgcn_ballot_w64(!x.finite()) == 0) {
    accumulate<D>(acc, x, w);
    return;
  }
  using M = ColMap<D>;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const float wj = __shfl(w[j & 3], (j >> 2) * 16 + i, 64);
    if (row0 + j >= S || !allowed(j, i)) continue;
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        acc[db][r] = fmaf(wj, X[(size_t)(row0 + j) * ld + M::d_of(db / M::VW, 4 * g + r) + db % M::VW], acc[db][r]);
  }
}
// this wave's transposed accumulator -> LDS as [column][D], rows of D + 4 floats
template <int D> __device__ __forceinline__ void stage_acc(float* dst, const f32x4 (&acc)[D / 16], int g, int i) {
  using M = ColMap<D>;
  typedef float vec __attribute__((ext_vector_type(M::VW)));
#pragma unroll
  for (int gr = 0; gr < M::NG; ++gr)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      vec x;
#pragma unroll
      for (int e = 0; e < M::VW; ++e) x[e] = acc[gr * M::VW + e][r];
      *reinterpret_cast<vec*>(dst + i * (D + 4) + M::d_of(gr, 4 * g + r)) = x;
    }
}
// thread -> its D/16 elements of column threadIdx.x/16, in pieces of W
template <int D> struct Share {
  static constexpr int W = D == 32 ? 2 : 4, N = D / 16 / W;
  typedef float vec __attribute__((ext_vector_type(W)));
  static __device__ __forceinline__ int d_of(int p) { return (p * 16 + (threadIdx.x & 15)) * W; }
};

template <int D>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(const float* __restrict__ qkv, float* __restrict__ out,
                                                           float* __restrict__ lse, int S, int a) {
  constexpr int NB = D / 16;
  __shared__ __attribute__((aligned(16))) float part[4 * 16 * (D + 4)];
  __shared__ float stat[2][4][16];   // maximum and sum of each wave and query
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, g = lane >> 4;
  const int P = a * D, n = blockIdx.y, b = blockIdx.z;
  const size_t ld = 3 * (size_t)P;
  const float* base = qkv + (size_t)b * S * ld + (size_t)n * D;
  const int qb = gridDim.x - 1 - blockIdx.x;   // the rows with most keys start first
  const float c = kLog2e / sqrtf((float)D);

  RowFrag<D> q;
  q.load(base, ld, qb * 16 + i, S, g);
  f32x4 o[NB];
#pragma unroll
  for (int db = 0; db < NB; ++db) o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = kNoKey, l = 0.f;
  auto block = [&](const RowFrag<D>& k, const ColFrag<D>& v, int kb, auto diag) {
    f32x4 s = rows_times_cols<D>(k, q) * c;
    if constexpr (decltype(diag)::value) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * g + r > i) s[r] = -INFINITY;
    }
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), alpha = __builtin_amdgcn_exp2f(m - mn);
    f32x4 p;
    l *= alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __builtin_amdgcn_exp2f(s[r] - mn);
      l += p[r];
    }
#pragma unroll
    for (int db = 0; db < NB; ++db) o[db] *= alpha;
    m = mn;
    if constexpr (decltype(diag)::value)
      accumulate_diagonal<D>(o, v, p, base + 2 * P, ld, kb * 16, S, g, i, [](int key, int query) { return key <= query; });
    else
      accumulate<D>(o, v, p);
  };
  RowFrag<D> k;
  if (wave <= qb) k.load(base + P, ld, wave * 16 + i, S, g);
  for (int kb = wave; kb <= qb; kb += 4) {
    ColFrag<D> v;
    v.load(base + 2 * P, ld, kb * 16, S, g, i);
    RowFrag<D> kn = k;
    if (kb + 4 <= qb) kn.load(base + P, ld, (kb + 4) * 16 + i, S, g);   // the next block's keys, ahead of their use
    if (kb == qb) block(k, v, kb, std::true_type{});
    else block(k, v, kb, std::false_type{});
    k = kn;
  }

  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  stage_acc<D>(part + wave * 16 * (D + 4), o, g, i);
  if (g == 0) {
    stat[0][wave][i] = m;
    stat[1][wave][i] = l;
  }
  __syncthreads();
  const int col = threadIdx.x >> 4, row = qb * 16 + col;
  if (row >= S) return;
  float mt = stat[0][0][col], lt = 0.f, f[4];
#pragma unroll
  for (int w = 1; w < 4; ++w) mt = fmaxf(mt, stat[0][w][col]);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    f[w] = __builtin_amdgcn_exp2f(stat[0][w][col] - mt);
    lt += f[w] * stat[1][w][col];
  }
  const float inv = 1.f / lt;
  using Sh = Share<D>;
#pragma unroll
  for (int p = 0; p < Sh::N; ++p) {
    typename Sh::vec v = f[0] * *reinterpret_cast<const typename Sh::vec*>(part + col * (D + 4) + Sh::d_of(p));
#pragma unroll
    for (int w = 1; w < 4; ++w) v += f[w] * *reinterpret_cast<const typename Sh::vec*>(part + (w * 16 + col) * (D + 4) + Sh::d_of(p));
    *reinterpret_cast<typename Sh::vec*>(out + ((size_t)b * S + row) * P + (size_t)n * D + Sh::d_of(p)) = v * inv;
  }
  if ((threadIdx.x & 15) == 0) lse[((size_t)b * a + n) * S + row] = (mt + __builtin_amdgcn_logf(lt)) * kLn2;
}

// The waves' partial sums of one transposed result -> rows of dst (16 from row0), in fixed order
template <int D>
__device__ __forceinline__ void reduce_and_store(float* part, const f32x4 (&acc)[D / 16], float* dst, size_t ld, int row0, int S,
                                                 int wave, int g, int i) {
  stage_acc<D>(part + wave * 16 * (D + 4), acc, g, i);
  __syncthreads();
  const int col = threadIdx.x >> 4;
  using Sh = Share<D>;
  if (row0 + col < S)
#pragma unroll
    for (int p = 0; p < Sh::N; ++p) {
      typename Sh::vec v = *reinterpret_cast<const typename Sh::vec*>(part + col * (D + 4) + Sh::d_of(p));
#pragma unroll
      for (int w = 1; w < 4; ++w) v += *reinterpret_cast<const typename Sh::vec*>(part + (w * 16 + col) * (D + 4) + Sh::d_of(p));
      *reinterpret_cast<typename Sh::vec*>(dst + (size_t)(row0 + col) * ld + Sh::d_of(p)) = v;
    }
}

// grid.x = 2 * blocks: even indices dQ of a query block, odd ones dK and dV of a key block, each
// kind's longest first
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_f32_kernel(const float* __restrict__ qkv, const float* __restrict__ out,
                                                           const float* __restrict__ lse, const float* __restrict__ dout,
                                                           float* __restrict__ dqkv, int S, int a) {
  constexpr int NB = D / 16;
  __shared__ __attribute__((aligned(16))) float part[4 * 16 * (D + 4)];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, g = lane >> 4;
  const int P = a * D, n = blockIdx.y, b = blockIdx.z;
  const size_t ld = 3 * (size_t)P;
  const float* base = qkv + (size_t)b * S * ld + (size_t)n * D;
  const float* obase = out + (size_t)b * S * P + (size_t)n * D;
  const float* dobase = dout + (size_t)b * S * P + (size_t)n * D;
  float* dbase = dqkv + (size_t)b * S * ld + (size_t)n * D;
  const float* lse_h = lse + ((size_t)b * a + n) * S;
  const float scale = 1.f / sqrtf((float)D), c = kLog2e / sqrtf((float)D);
  const int nb = (S + 15) / 16;
  // sum over d of x o y for row i of the two fragments: the same on all lanes of the row
  auto row_dot = [&](const RowFrag<D>& x, const RowFrag<D>& y) {
    f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < NB; ++q) t += x.v[q] * y.v[q];
    float s = (t[0] + t[1]) + (t[2] + t[3]);
    s += __shfl_xor(s, 16, 64);
    return s + __shfl_xor(s, 32, 64);
  };
  if ((blockIdx.x & 1) == 0) {
    const int qb = nb - 1 - (int)(blockIdx.x >> 1), row = qb * 16 + i;
    RowFrag<D> q, dO, oo;
    q.load(base, ld, row, S, g);
    dO.load(dobase, P, row, S, g);
    oo.load(obase, P, row, S, g);
    const float delta = row_dot(dO, oo), L2 = lse_h[row < S ? row : 0] * kLog2e;
    f32x4 dq[NB];
#pragma unroll
    for (int db = 0; db < NB; ++db) dq[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kb = wave; kb <= qb; kb += 4) {
      RowFrag<D> k, v;
      ColFrag<D> kc;
      k.load(base + P, ld, kb * 16 + i, S, g);
      v.load(base + 2 * P, ld, kb * 16 + i, S, g);
      kc.load(base + P, ld, kb * 16, S, g, i);
      const f32x4 s = rows_times_cols<D>(k, q), dp = rows_times_cols<D>(v, dO);
      f32x4 ds;
#pragma unroll
      for (int r = 0; r < 4; ++r) ds[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c, -L2)) * (dp[r] - delta) * scale;
      if (kb == qb) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (4 * g + r > i) ds[r] = 0.f;
        accumulate_diagonal<D>(dq, kc, ds, base + P, ld, kb * 16, S, g, i, [](int key, int query) { return key <= query; });
      } else {
        accumulate<D>(dq, kc, ds);
      }
    }
    reduce_and_store<D>(part, dq, dbase, ld, qb * 16, S, wave, g, i);
  } else {
    const int kb = blockIdx.x >> 1;
    RowFrag<D> k, v;
    k.load(base + P, ld, kb * 16 + i, S, g);
    v.load(base + 2 * P, ld, kb * 16 + i, S, g);
    f32x4 dk[NB], dv[NB];
#pragma unroll
    for (int db = 0; db < NB; ++db) dk[db] = dv[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int qb = kb + wave; qb < nb; qb += 4) {
      RowFrag<D> q, dO, oo;
      ColFrag<D> qc, doc;
      q.load(base, ld, qb * 16 + i, S, g);
      dO.load(dobase, P, qb * 16 + i, S, g);
      oo.load(obase, P, qb * 16 + i, S, g);
      qc.load(base, ld, qb * 16, S, g, i);
      doc.load(dobase, P, qb * 16, S, g, i);
      const float delta_row = row_dot(dO, oo);   // of query i; this lane needs those of queries 4g + r
      const f32x4 s = rows_times_cols<D>(q, k), dp = rows_times_cols<D>(dO, v);
      f32x4 p, ds;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = qb * 16 + 4 * g + r;
        const float L2 = lse_h[row < S ? row : 0] * kLog2e;
        const float delta = __shfl(delta_row, 4 * g + r, 64);   // with every lane active: lanes read each other
        const bool counts = row < S && (qb != kb || 4 * g + r >= i);
        p[r] = counts ? __builtin_amdgcn_exp2f(fmaf(s[r], c, -L2)) : 0.f;
        ds[r] = counts ? p[r] * (dp[r] - delta) * scale : 0.f;
      }
      if (qb == kb) {
        auto allowed = [](int query, int key) { return query >= key; };
        accumulate_diagonal<D>(dv, doc, p, dobase, P, qb * 16, S, g, i, allowed);
        accumulate_diagonal<D>(dk, qc, ds, base, ld, qb * 16, S, g, i, allowed);
      } else {
        accumulate<D>(dv, doc, p);
        accumulate<D>(dk, qc, ds);
      }
    }
    reduce_and_store<D>(part, dk, dbase + P, ld, kb * 16, S, wave, g, i);
    __syncthreads();   // every thread has read dK's partial sums
    reduce_and_store<D>(part, dv, dbase + 2 * P, ld, kb * 16, S, wave, g, i);
  }
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

template <int D> hipError_t fwd_d(int B, int S, int a, const float* qkv, float* out, float* lse, hipStream_t st) {
  hipLaunchKernelGGL(attn_fwd_f32_kernel<D>, dim3((S + 15) / 16, a, B), dim3(256), 0, st, qkv, out, lse, S, a);
  return hipGetLastError();
}
template <int D>
hipError_t bwd_d(int B, int S, int a, const float* qkv, const float* out, const float* lse, const float* dout, float* dqkv, hipStream_t st) {
  hipLaunchKernelGGL(attn_bwd_f32_kernel<D>, dim3(2 * ((S + 15) / 16), a, B), dim3(256), 0, st, qkv, out, lse, dout, dqkv, S, a);
  return hipGetLastError();
}

}  // namespace

bool attention_f32_supported(const void* qkv, const void* out, const void* dout, const void* dqkv) {
  return aligned16(qkv) && aligned16(out) && aligned16(dout) && aligned16(dqkv);
}

hipError_t attention_fwd_f32(int B, int S, int a, int d, const void* qkv, void* out, float* lse, hipStream_t st) {
  const float* q = (const float*)qkv;
  switch (d) {
    case 32: return fwd_d<32>(B, S, a, q, (float*)out, lse, st);
    case 64: return fwd_d<64>(B, S, a, q, (float*)out, lse, st);
    case 128: return fwd_d<128>(B, S, a, q, (float*)out, lse, st);
  }
  return hipErrorInvalidValue;
}
hipError_t attention_bwd_f32(int B, int S, int a, int d, const void* qkv, const void* out, const float* lse,
                             const void* dout, void* dqkv, hipStream_t st) {
  const float *q = (const float*)qkv, *o = (const float*)out, *g = (const float*)dout;
  switch (d) {
    case 32: return bwd_d<32>(B, S, a, q, o, lse, g, (float*)dqkv, st);
    case 64: return bwd_d<64>(B, S, a, q, o, lse, g, (float*)dqkv, st);
    case 128: return bwd_d<128>(B, S, a, q, o, lse, g, (float*)dqkv, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace gpts

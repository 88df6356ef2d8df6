// The fixed-order reduction of partial column sums as device code, for its own kernel and for the workgroups that
// launches of weight gradients have over (gemm_tiles.hpp, gemm_f32.hip).
#pragma once
#include "kernels.hpp"

namespace gpts {

// For every segment: out[c] += sum_{g<G} partial[g*stride + c], c < N, see ReduceSeg.  32 columns x
// 32 row groups per workgroup, four columns per load; the row groups are combined through LDS in fixed
// order, so the result is deterministic.  One launch takes all the bias and LayerNorm gradients of a
// layer: each is a few microseconds of launch and latency whatever its size (16 rows: 2.4 us).
// NS: segments there is room for.  One alone has a form of its own, without the search and with a sixth of
// the arguments: 0.3 us less to launch.
// NB: micro-batches there is room for.  Their loads go out together, and each one's row groups are added by 32
// threads of its own, before the eight sums are added to out in order: the same sums as one micro-batch after the
// other, which waited for memory and two barriers each time: eight times 64 rows of partial sums 9.9 -> 4.7 us (with three such
// launches a layer and window, 4 chunks of width 1024, 8 micro-batches of 512 tokens 2328 -> 2265 us; two are left where the late
// sums have room beside each other).
template <int NS> struct ReduceArgs {
  ReduceSeg seg[NS];
  int first[NS];   // first workgroup of a segment
};
// 256 threads; block: the workgroup's place among those of the segments; sm: its LDS
template <int NS, int NB> __device__ __forceinline__ void reduce_columns(const ReduceArgs<NS>& args, int block, float (*sm)[32][33]) {
  static_assert(NB == 1 || NB * 32 == 256, "32 threads per micro-batch");
  int k = 0;
#pragma unroll
  for (int i = 1; i < NS; ++i)
    if (block >= args.first[i]) k = i;
  const ReduceSeg& sg = args.seg[k];
  const int col0 = (block - args.first[k]) * 32;
  const int cq = threadIdx.x & 7, ry = threadIdx.x >> 3, c4 = col0 + cq * 4;
  const int cl = threadIdx.x & 31, bt = threadIdx.x >> 5, c = col0 + cl;   // NB > 1: column and micro-batch of the sums
  const bool adds = threadIdx.x < 32 && c < sg.N;
  float* const out = c < sg.n0 ? sg.out0 + c : (c < sg.n1 ? sg.out1 + (c - sg.n0) : sg.out2 + (c - sg.n1));
  float total = adds ? *out : 0.f;
  const int n = NB == 1 ? 1 : sg.batch;
  const size_t next = (size_t)sg.G * sg.stride;      // between micro-batches
  constexpr int UNROLL = NB == 1 ? 4 : 2;
  f32x4 s[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) s[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (c4 < sg.N) {
    const float* const p = sg.partial + c4;
#pragma unroll UNROLL
    for (int g = ry; g < sg.G; g += 32) {
      f32x4 v[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) v[b] = *reinterpret_cast<const f32x4*>(p + (b < n ? b : 0) * next + (size_t)g * sg.stride);
#pragma unroll
      for (int b = 0; b < NB; ++b) s[b] += v[b];
    }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) sm[b][ry][cq * 4 + e] = s[b][e];
  __syncthreads();
  if (NB > 1 || adds) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 32; ++i) t += sm[NB > 1 ? bt : 0][i][cl];
    if constexpr (NB == 1) total += t;
    else sm[bt][0][cl] = t;    // (only this thread reads column cl of its micro-batch)
  }
  if constexpr (NB > 1) {
    __syncthreads();
    if (adds) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (b < n) total += sm[b][0][cl];
    }
  }
  if (adds) *out = total;
}

// The segments' places in a launch; returns how many workgroups they take.
template <int NS> inline int reduce_layout(const ReduceSeg* segs, int n, ReduceArgs<NS>* a) {
  int blocks = 0;
  for (int i = 0; i < NS; ++i) {
    a->first[i] = i < n ? blocks : 0x7fffffff;      // (never reached)
    if (i >= n) continue;
    a->seg[i] = segs[i];
    blocks += (segs[i].N + 31) / 32;
  }
  return blocks;
}

// what a launch of weight gradients takes: up to kMaxReduceSegs, each of one micro-batch
inline bool few_sums(const ReduceSeg* segs, int n) {
  if (n < 0 || n > kMaxReduceSegs) return false;
  for (int i = 0; i < n; ++i)
    if (segs[i].batch != 1) return false;
  return true;
}

}  // namespace gpts

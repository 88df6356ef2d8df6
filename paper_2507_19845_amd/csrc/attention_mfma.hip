// Causal softmax attention on the gfx950 matrix cores (bf16 in, fp32 accumulate).
//
// Forward, per (batch, head): a workgroup owns 128 (or, two waves to 32 rows, 64) query rows and
// walks the key/value rows in tiles of 64 up to the diagonal with an online
// softmax.  Both products are computed TRANSPOSED so that no value ever has to
// move between lanes:
//   S^T[key][query] = K Q^T      A-operand = K fragment (ds_read_b128 from the
//                                K tile), B-operand = Q fragment (registers)
//   O^T[d][query]   = V^T P^T    A-operand = V^T fragment, B-operand = P^T, which
//                                is exactly the S^T accumulator of the same lane,
//                                rounded to bf16.
// A lane therefore owns one query column throughout: its running max, running
// sum and the rescaling of O are per-lane scalars; only the max needs one
// exchange with the lane that holds the other half of the keys (lane ^ 32).
//
// Every product that contracts over the sequence index (O^T = V^T P^T, and in the
// backward pass dV^T = dO^T P, dK^T = Q^T dS, dQ^T = K^T dS^T) needs its A operand
// with the sequence index running fastest.  The transposing LDS read (ds_read_b64_tr_b16) delivers that from the
// same row-major tile the other products read.  At D = 64 and 128 it has two-way bank conflicts (swz16()), and these
// are 0.21 to 0.33 of the LDS's active time, but the LDS is active for at most 0.41 of a kernel's: a tile is copied once and
// read both ways.  (Transposed copies of V, Q, K and dO, written to memory by
// a kernel of their own and streamed beside the row-major tiles, were the form before: B x S x heads x D,
// forward and backward, us: 1x8191x16x128 297 + 942, now 287 + 858; 1x2048x16x128 44.5 + 97, now 38 + 86;
// 16x333x12x32 12.5 + 32.9, now 7.9 + 24.6.)
// K, V, Q and dO tiles go global -> LDS by DMA, double buffered.
#include <type_traits>

#include "kernels.hpp"

namespace gpts {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Wave priority inside the kernels: raised around a run of matrix instructions, so that of the
// two waves sharing a SIMD the one feeding the matrix pipe issues first and the other's softmax
// arithmetic fills the gaps (measured: forward +1.7 %, backward +1 %).
#define GPTS_PRIO(p) __builtin_amdgcn_s_setprio(p)

constexpr int BKV = 64;   // rows per streamed tile
// Stands for "no key seen yet" in the running maximum: no finite logit is smaller, and the difference of
// two such values is 0 and not NaN.  (A wave's share of a row's keys may have no logit but -inf.)
constexpr float kNoKey = -3.4028234663852886e38f;

// A [64][D] tile lies in LDS as panels of up to 64 columns, [64][PW] each (constant offsets between them, and fewer
// addresses to keep), with the 16-byte chunks of a panel row XOR-swizzled with the row.  A 16-byte LDS read serves 16
// lanes at a time over the 64 banks, lanes {0-3, 12-15, 20-27} of a half wave, then its others; a half wave
// reads one chunk of 32 rows, and the rows of each such group land in 16 different places.  A transposing read serves a
// half wave at a time, four chunks of four rows r .. r+3: at D = 32, rows of 64 bytes, in different banks; in rows of 128
// bytes r and r+2 start at the same bank, and the swizzle moves chunks 0-3 of both within the same 64 bytes, so half of the
// banks are used twice.
template <int D> constexpr int kPanel = D < 64 ? D : 64;            // columns of a panel
template <int D> constexpr int kPanelBytes = BKV * kPanel<D> * 2;
template <int D> __device__ __forceinline__ int swz16(int row) { return D == 32 ? (row >> 2) & 3 : (row >> 1) & 7; }

// Eight accumulator values rounded to 16 bits as the next product's operand.  All operand
// registers are typed bf16x8; with F16 they hold fp16 bits (forward activations kept in fp16).
template <bool F16 = false> __device__ __forceinline__ bf16x8 pack8(const f32x16& v, int base) {
  if constexpr (F16) {
    f16x8 r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (f16)v[base + e];
    return __builtin_bit_cast(bf16x8, r);
  } else {
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (bf16)v[base + e];
    return r;
  }
}
// acc += A (32 x 16) * B (16 x 32); F16: the operand registers hold fp16 values
template <bool F16 = false>
__device__ __forceinline__ f32x16 mma32(const bf16x8& a, const bf16x8& b, const f32x16& acc) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), acc, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}

// Marks a register value as used.  The tiles travel by DMA instructions the compiler
// does not track, while ordinary global loads it does track are waited for with
// "s_waitcnt vmcnt(n)" in front of their first use.  If that first use sits inside the
// tile loop, the wait stays there in every iteration and -- the counter being shared --
// also drains the next tile's DMA, which removes the double buffering.  Using the loaded
// registers once before the loop moves the wait in front of the loop.
__device__ __forceinline__ void settle(const bf16x8& v) {
  asm volatile("" ::"v"(__builtin_bit_cast(i32x4, v)));
}
__device__ __forceinline__ void settle(float v) { asm volatile("" ::"v"(v)); }

template <typename P> __device__ __forceinline__ P* after(P* p, size_t bytes) {
  return (P*)((const char*)p + bytes);   // (by way of an integer it would no longer count as global memory)
}
// blockIdx.y counts the B sequences of every micro-batch; stride 0: there is one (and no division)
__device__ __forceinline__ int microbatch(int B, size_t stride) {
  return stride ? __builtin_amdgcn_readfirstlane(blockIdx.y / B) : 0;
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(size_t)(__attribute__((address_space(3))) const char*)p;
}

// One DMA instruction: lane i copies 16 bytes from src + off_i to LDS dst + 16*i.
// Inline assembly on purpose (see settle()): the kernels wait for these copies
// explicitly (s_waitcnt vmcnt(0)) before the barrier that publishes a tile.
__device__ __forceinline__ void dma16(const void* src, uint32_t off, uint32_t dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(src) : "memory");
}
// 64 floats global -> LDS by one DMA instruction of one wave (lane i: src[idx_i] -> dst[i])
__device__ __forceinline__ void dma_floats(const float* __restrict__ src, int idx, float* dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_addr(dst)), "v"((uint32_t)idx * 4u), "s"(src) : "memory");
}

// 64 rows starting at global row `row0` (clamped to < S) are copied by the NW waves
// of the workgroup; each DMA instruction moves 1 KiB (a tile of fewer instructions than waves
// is copied by the first waves only).
template <int D, int NW>
__device__ __forceinline__ void dma_tile(const bf16* __restrict__ src, size_t ld, int row0, int S,
                                         char* tile, int wave, int lane) {
  constexpr int CPR = kPanel<D> / 8;           // chunks per panel row
  constexpr int NT = BKV * D * 2 / 1024;       // instructions per tile
  constexpr int NI = NT >= NW ? NT / NW : 1;   // instructions per (issuing) wave
  static_assert(NT >= 1 && (NT >= NW ? NT % NW == 0 : true), "tile / wave count mismatch");
  if (NT < NW && wave >= NT) return;
  const uint32_t lds_tile = lds_addr(tile);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int slot = (wave * NI + i) * 64 + lane;
    const int r = slot / CPR % BKV, pc = slot % CPR;
    const int c = slot / (CPR * BKV) * CPR + (pc ^ swz16<D>(r));
    int gr = row0 + r;
    gr = gr < S ? gr : S - 1;
    dma16(src, (uint32_t)(((size_t)gr * ld + c * 8) * 2), lds_tile + (wave * NI + i) * 1024);
  }
}
// Rows from `first` on of a tile in LDS set to zero: the rows past the sequence's end, which the copy
// filled with its last row.  The caller puts a barrier behind it.
template <int D, int NW> __device__ __forceinline__ void zero_rows(char* tile, int first, int wave, int lane) {
  constexpr int CPR = kPanel<D> / 8;
  for (int i = wave * 64 + lane; i < BKV * D / 8; i += NW * 64)
    if (i / CPR % BKV >= first) *reinterpret_cast<f32x4*>(tile + i * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
}

// delta[b][n][s] = sum_d dO * O: one row of a head per D/8 lanes.
template <int D, bool O16>
__global__ __launch_bounds__(256) void attn_delta_kernel(const bf16* __restrict__ out0, const bf16* __restrict__ dout0,
                                                         float* __restrict__ delta0, int S, int a, int total, size_t stride) {
  const bf16* const out = after(out0, blockIdx.y * stride);
  const bf16* const dout = after(dout0, blockIdx.y * stride);
  float* const delta = after(delta0, blockIdx.y * stride);
  constexpr int TPR = D / 8;
  const int t = (int)(blockIdx.x * 256 + threadIdx.x);
  const int i = t / TPR, cc = t % TPR;     // i: [b][s][n], as the rows lie in memory
  float acc = 0.f;
  if (i < total) {
    const bf16x8 o = *reinterpret_cast<const bf16x8*>(out + (size_t)i * D + cc * 8);
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(dout + (size_t)i * D + cc * 8);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fmaf(O16 ? (float)__builtin_bit_cast(f16x8, o)[e] : (float)o[e], (float)v[e], acc);
  }
#pragma unroll
  for (int x = TPR / 2; x > 0; x >>= 1) acc += __shfl_xor(acc, x, 64);
  if (cc == 0 && i < total) {
    const int n = i % a, bs = i / a, b = bs / S, row = bs % S;
    delta[((size_t)b * a + n) * S + row] = acc;
  }
}

// Fragment whose contraction runs over the tile's rows (A operand, 32 columns d x 16 rows), by two transposing
// reads: lane (d, h) gets rows 4h .. +3 and 8 + 4h .. +3 of the group of 16, the order in which an MFMA accumulator
// hands out its rows, so the accumulator of the other factor is the B operand as it is.  tr_off(): the lane's byte
// offset for columns 0-31 and row group 0; columns 32 db .. and the second read (8 rows on) XOR and add constants.
template <int D> __device__ __forceinline__ int tr_off(int lane) {
  const int h = lane >> 5, cb = (lane >> 4) & 1, q = (lane & 15) >> 2, p = lane & 3, r = 4 * h + q;
  return r * (kPanel<D> * 2) + (((2 * cb + (p >> 1)) ^ swz16<D>(r)) << 4) + (p & 1) * 8;
}
typedef short s16x4 __attribute__((ext_vector_type(4)));
template <int D> __device__ __forceinline__ bf16x8 tr_frag(const char* tile, int off, int group, int db) {
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  typedef s16x4 __attribute__((address_space(3)))* lds_p;
  constexpr int RB = kPanel<D> * 2, flip = D == 32 ? 32 : 64;   // flip: swz16(row + 8) ^ swz16(row), in bytes
  const char* p = tile + (db >> 1) * kPanelBytes<D> + group * 16 * RB;
  // (off has no bit of 64 for panels of 128 bytes: what is XORed there is an added constant)
  const int x = (db & 1) * 64;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p + (D == 32 ? off : off + x)));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p + 8 * RB + (D == 32 ? off ^ flip : off + (x ^ flip))));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// Fragment whose contraction runs over the tile's columns (A operand, 32 rows x 16 d), one 16-byte read: row block rb
// (32 rows), k-step kk.
template <int D> __device__ __forceinline__ int natural_off(int ql, int h) {
  return ql * (kPanel<D> * 2) + ((h ^ swz16<D>(ql)) << 4);
}
template <int D> __device__ __forceinline__ bf16x8 natural_frag(const char* tile, int off, int rb, int kk) {
  constexpr int KP = kPanel<D> / 16;
  return *reinterpret_cast<const bf16x8*>(tile + kk / KP * kPanelBytes<D> + rb * 32 * (kPanel<D> * 2) + (off ^ (kk % KP << 5)));
}

// element e of 16 bf16 values: an operation on the packed pair, where a conversion would first take it apart
__device__ __forceinline__ float element_of(const bf16x8 (&v)[2], int e) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  const unsigned w = __builtin_bit_cast(u32x4, v[e >> 3])[(e & 7) >> 1];
  return __builtin_bit_cast(float, e & 1 ? w & 0xffff0000u : w << 16);
}

template <int... I, class F> __device__ __forceinline__ void static_for_seq(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(F&& f) { static_for_seq(std::make_integer_sequence<int, N>{}, f); }

// the larger of a lane's value and that of lane ^ 32
__device__ __forceinline__ float max_of_halves(float v) {
  const unsigned x = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  const unsigned lo = r[0], hi = r[1];   // (a bit cast of r[1] itself gives r[0]'s)
  return fmaxf(__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi));
}
// The order asked of the compiler for N matrix instructions and what goes between them: LDS reads (NL for each) AHEAD
// instructions before their use, NV vector instructions after each of the first LEAD and then NW with one or two exponentials.
template <int N, int NL, int AHEAD, int LEAD, int NV, int NW, int I = 0> __device__ __forceinline__ void interleave() {
  if constexpr (I == 0) __builtin_amdgcn_sched_group_barrier(0x100, AHEAD * NL, 0);
  if constexpr (I < N) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if constexpr (I + AHEAD < N) __builtin_amdgcn_sched_group_barrier(0x100, NL, 0);
    if constexpr (I < LEAD) {
      __builtin_amdgcn_sched_group_barrier(0x002, NV, 0);
    } else {
      __builtin_amdgcn_sched_group_barrier(0x002, NW, 0);
      __builtin_amdgcn_sched_group_barrier(0x400, 1 + (I & 1), 0);
    }
    interleave<N, NL, AHEAD, LEAD, NV, NW, I + 1>();
  }
}

// ---- forward -----------------------------------------------------------------------------
// grid (heads, batch, query tiles): the heaviest query tiles of all heads start first.
// F16: qkv, the probabilities and out are fp16 (same layouts, f16 instructions).
// RW x SW waves: RW blocks of 32 queries (4, 8 for many long sequences); with SW = 2 a second wave per block takes the other 32 keys
// of every tile, and the two running maxima, sums and outputs are merged through LDS at the end.
template <int D, bool F16, int RW, int SW>
__global__ __launch_bounds__(64 * RW * SW, 2) void attn_fwd_mfma_kernel(const bf16* __restrict__ qkv0, bf16* __restrict__ out0,
                                                               float* __restrict__ lse0, int S, int a, int B, size_t stride) {
  constexpr int KSTEPS = D / 16;   // MFMA k-steps over the head dimension
  constexpr int DB = D / 32;       // 32-row blocks of O^T
  constexpr int TILE = BKV * D * 2;  // bytes of one K or V tile
  constexpr int NW = RW * SW, BQ = 32 * RW, NKB = 2 / SW;        // queries; 32-key blocks of a tile per wave
  __shared__ __attribute__((aligned(1024))) char lds[4 * TILE];  // [stage][K | V]

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rw = wave % RW, kb0 = wave / RW * NKB;   // this wave's query block; its first key block of a tile
  const int qt = gridDim.z - 1 - blockIdx.z;
  const int n = blockIdx.x, mb = microbatch(B, stride), b = blockIdx.y - mb * B;   // head; micro-batch, sequence
  const bf16* __restrict__ qkv = after(qkv0, mb * stride);
  bf16* __restrict__ out = after(out0, mb * stride);
  float* __restrict__ lse = after(lse0, mb * stride);
  const int P = a * D;
  const size_t ld = 3 * (size_t)P;
  const bf16* base = qkv + (size_t)b * S * ld + (size_t)n * D;
  const int q0 = qt * BQ;
  const int ql = lane & 31, h = lane >> 5;
  const int qrow = q0 + rw * 32 + ql;          // this lane's query
  const int qclamp = qrow < S ? qrow : S - 1;
  const int qmax_wave = min(q0 + rw * 32 + 31, S - 1);

  // Q fragments (B operand: column = query, 8 consecutive d per lane and k-step)
  bf16x8 qf[KSTEPS];
#pragma unroll
  for (int kk = 0; kk < KSTEPS; ++kk)
    qf[kk] = *reinterpret_cast<const bf16x8*>(base + (size_t)qclamp * ld + kk * 16 + h * 8);
#pragma unroll
  for (int kk = 0; kk < KSTEPS; ++kk) settle(qf[kk]);

  f32x16 oacc[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[i][e] = 0.f;
  float m_run = kNoKey, l_run = 0.f;
  const float c = 1.4426950408889634f / sqrtf((float)D);  // log2(e)/sqrt(D)

  const int koff = natural_off<D>(ql, h);
  const int voff = tr_off<D>(lane);

  const int last_key = min(q0 + BQ, S);               // keys [0, last_key) are needed
  const int nkv = (last_key + BKV - 1) / BKV;
  if constexpr (RW == 8) {
    // The logits of tile kt + 1 are formed while the softmax of tile kt is computed, matrix and vector instructions
    // alternating within the wave, and K runs a tile ahead of V: with eight waves behind one barrier a SIMD's two waves are in
    // the same phase, and one after the other the phases left its pipes idle in turn (1x8191x16x128 292 | 281 us; in
    // four waves, whose workgroups drift apart, it gains nothing: 300 | 308).
    f32x16 sacc[2][NKB];
    auto kbuf = [&](int i) -> char* { return lds + i * 2 * TILE; };
    auto vbuf = [&](int i) -> char* { return lds + i * 2 * TILE + TILE; };
    auto logits = [&](f32x16(&s)[NKB], const char* tK) {   // S^T = K Q^T for the wave's 32-key blocks
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
        for (int e = 0; e < 16; ++e) s[kb][e] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) s[kb] = mma32<F16>(natural_frag<D>(tK, koff, kb0 + kb, kk), qf[kk], s[kb]);
      }
    };
    dma_tile<D, NW>(base + P, ld, 0, S, kbuf(0), wave, lane);
    dma_tile<D, NW>(base + 2 * P, ld, 0, S, vbuf(0), wave, lane);
    if (nkv > 1) dma_tile<D, NW>(base + P, ld, BKV, S, kbuf(1), wave, lane);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (kb0 * 32 <= qmax_wave) logits(sacc[0], kbuf(0));

    auto tile = [&](auto cur_c, int kt) {
      constexpr int cur = decltype(cur_c)::value, nxt = cur ^ 1;
      f32x16(&s)[NKB] = sacc[cur];
      // K(kt + 1) and V(kt) have landed; K(kt) and V(kt - 1) are done with
      asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      const int k0 = kt * BKV;
      if (kt + 2 < nkv) dma_tile<D, NW>(base + P, ld, k0 + 2 * BKV, S, kbuf(cur), wave, lane);
      if (kt + 1 < nkv) dma_tile<D, NW>(base + 2 * P, ld, k0 + BKV, S, vbuf(nxt), wave, lane);
      if (k0 + BKV > S) {   // (uniform) keys past the last one: p = 0 has to meet v = 0
        zero_rows<D, NW>(vbuf(cur), S - k0, wave, lane);
        __syncthreads();
      }
      const int kw0 = k0 + kb0 * 32;
      if (kw0 > qmax_wave) return;  // every key of this tile is masked for this wave
      float m_new, mc, psum = 0.f;
      auto maximum = [&]() {
        float mx = s[0][0];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
          for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[kb][e]);
        m_new = fmaxf(m_run, max_of_halves(mx));
        mc = m_new * c;
      };
      bf16x8 pf[2 * NKB];
      auto probabilities = [&](int ks) {     // 16 keys
#pragma unroll
        for (int e = (ks & 1) * 8; e < (ks & 1) * 8 + 8; ++e) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[ks >> 1][e], c, -mc));
          s[ks >> 1][e] = p;
          psum += p;
        }
        pf[ks] = pack8<F16>(s[ks >> 1], (ks & 1) * 8);
      };
      // (a tile that the diagonal crosses is the wave's last: blocks of 32 queries, keys at multiples of 32)
      if (kt + 1 < nkv && kw0 + BKV <= qmax_wave) {
        logits(sacc[nxt], kbuf(nxt));
        maximum();
#pragma unroll
        for (int ks = 0; ks < NKB; ++ks) probabilities(ks);
        interleave<NKB * KSTEPS, 1, 1, KSTEPS / 2, 5, 4>();
      } else {
        if (kw0 + NKB * 32 - 1 > q0 + rw * 32) {
#pragma unroll
          for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const int key = kw0 + kb * 32 + (e >> 2) * 8 + h * 4 + (e & 3);
              if (key > qrow) s[kb][e] = -INFINITY;
            }
        }
        maximum();
#pragma unroll
        for (int ks = 0; ks < NKB; ++ks) probabilities(ks);
      }
      // the running maximum rarely moves after the first tiles: skip the rescaling of the
      // output accumulators when no lane of the wave needs it
      if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c);
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) oacc[i][e] *= alpha;
        m_run = m_new;
      }
      // ---- O^T += V^T P^T, the second half of the probabilities between the matrix instructions of the first
#pragma unroll
      for (int ks = NKB; ks < 2 * NKB; ++ks) probabilities(ks);
#pragma unroll
      for (int ks = 0; ks < 2 * NKB; ++ks)
#pragma unroll
        for (int db = 0; db < DB; ++db) oacc[db] = mma32<F16>(tr_frag<D>(vbuf(cur), voff, kb0 * 2 + ks, db), pf[ks], oacc[db]);
      interleave<2 * NKB * DB, 2, 2 * NKB * DB < 3 ? 2 * NKB * DB : 3, 0, 0, 4>();
      l_run += psum;
    };
    for (int kt = 0; kt < nkv; kt += 2) {
      tile(std::integral_constant<int, 0>{}, kt);
      if (kt + 1 < nkv) tile(std::integral_constant<int, 1>{}, kt + 1);
    }
  } else {
    dma_tile<D, NW>(base + P, ld, 0, S, lds, wave, lane);
    dma_tile<D, NW>(base + 2 * P, ld, 0, S, lds + TILE, wave, lane);

    for (int kt = 0; kt < nkv; ++kt) {
      asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      const int k0 = kt * BKV;
      const char* tK = lds + (kt & 1) * 2 * TILE;
      const char* tV = tK + TILE;
      if (kt + 1 < nkv) {
        char* nK = lds + ((kt + 1) & 1) * 2 * TILE;
        dma_tile<D, NW>(base + P, ld, k0 + BKV, S, nK, wave, lane);
        dma_tile<D, NW>(base + 2 * P, ld, k0 + BKV, S, nK + TILE, wave, lane);
      }
      if (k0 + BKV > S) {   // (uniform) keys past the last one: p = 0 has to meet v = 0
        zero_rows<D, NW>(lds + (kt & 1) * 2 * TILE + TILE, S - k0, wave, lane);
        __syncthreads();
      }
      const int kw0 = k0 + kb0 * 32;
      if (kw0 > qmax_wave) continue;  // every key of this tile is masked for this wave

      // ---- S^T = K Q^T for the wave's 32-key blocks ----------------------------------
      f32x16 sacc[NKB];
      if constexpr (SW == 1) GPTS_PRIO(1);
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
        for (int e = 0; e < 16; ++e) sacc[kb][e] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
          const bf16x8 kf = natural_frag<D>(tK, koff, kb0 + kb, kk);
          sacc[kb] = mma32<F16>(kf, qf[kk], sacc[kb]);
        }
      }
      if constexpr (SW == 1) GPTS_PRIO(0);
      // ---- causal mask (only tiles that reach past the first query of the wave) --------
      if (kw0 + NKB * 32 - 1 > q0 + rw * 32) {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int key = kw0 + kb * 32 + (e >> 2) * 8 + h * 4 + (e & 3);
            if (key > qrow) sacc[kb][e] = -INFINITY;
          }
      }
      // ---- online softmax ------------------------------------------------------------------
      float mx = sacc[0][0];
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sacc[kb][e]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m_run, mx);
      const float mc = m_new * c;
      float psum = 0.f;
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float p = __builtin_amdgcn_exp2f(fmaf(sacc[kb][e], c, -mc));
          sacc[kb][e] = p;
          psum += p;
        }
      // the running maximum rarely moves after the first tiles: skip the rescaling of the
      // output accumulators when no lane of the wave needs it
      if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c);
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) oacc[i][e] *= alpha;
        m_run = m_new;
      }
      l_run += psum;
      // ---- O^T += V^T P^T ------------------------------------------------------------------------
      if constexpr (SW == 1) GPTS_PRIO(1);
#pragma unroll
      for (int ks = 0; ks < 2 * NKB; ++ks) {     // 16 keys per step
        const bf16x8 pf = pack8<F16>(sacc[ks >> 1], (ks & 1) * 8);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const bf16x8 vf = tr_frag<D>(tV, voff, kb0 * 2 + ks, db);
          oacc[db] = mma32<F16>(vf, pf, oacc[db]);
        }
      }
      if constexpr (SW == 1) GPTS_PRIO(0);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // ---- finish: combine the two key halves' sums, normalise, store ------------------------
  float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if constexpr (SW == 2) {
    // the second wave of a query block hands its state over: outputs in the tile memory (every wave
    // has left the loop), maximum and sum beside it.  A wave that met no key, or no finite
    // logit, hands over kNoKey and zeros: it weighs 0 beside a finite maximum.
    __shared__ float ml[2][RW][kWave];
    __syncthreads();
    f32x4* ex = reinterpret_cast<f32x4*>(lds) + rw * (DB * 4 * kWave) + lane;
    if (kb0 != 0) {
#pragma unroll
      for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) ex[(i * 4 + g) * kWave] = f32x4{oacc[i][g * 4], oacc[i][g * 4 + 1], oacc[i][g * 4 + 2], oacc[i][g * 4 + 3]};
      ml[0][rw][lane] = m_run;
      ml[1][rw][lane] = l_tot;
    }
    __syncthreads();
    if (kb0 != 0) return;
    const float m2 = ml[0][rw][lane], m_new = fmaxf(m_run, m2);
    const float s1 = __builtin_amdgcn_exp2f((m_run - m_new) * c), s2 = __builtin_amdgcn_exp2f((m2 - m_new) * c);
    l_tot = l_tot * s1 + ml[1][rw][lane] * s2;
    m_run = m_new;
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 o2 = ex[(i * 4 + g) * kWave];
#pragma unroll
        for (int e = 0; e < 4; ++e) oacc[i][g * 4 + e] = oacc[i][g * 4 + e] * s1 + o2[e] * s2;
      }
  }
  if (qrow < S) {
    const float inv = 1.f / l_tot;
    bf16* orow = out + ((size_t)b * S + qrow) * P + (size_t)n * D;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if constexpr (F16) {
          f16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = sat_f16(oacc[db][g * 4 + e] * inv);
          *reinterpret_cast<f16x4*>(orow + db * 32 + g * 8 + h * 4) = o;
        } else {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16)(oacc[db][g * 4 + e] * inv);
          *reinterpret_cast<bf16x4*>(orow + db * 32 + g * 8 + h * 4) = o;
        }
      }
    if (h == 0) lse[((size_t)b * a + n) * S + qrow] = (m_run * c + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f;
  }
}


struct BwdArgs {
  const bf16 *qkv, *qk16, *dout, *out;   // out: where the query side forms delta, else null
  const float* lse;
  float* delta;
  bf16* dqkv;
  int S, a, B;           // B sequences per micro-batch
  size_t act, grad;      // bytes between the micro-batches' dqkv (grad) and everything else (act)
};
// the arguments of the workgroup's micro-batch mb
__device__ __forceinline__ BwdArgs at_microbatch(BwdArgs p, int mb) {
  p.qkv = after(p.qkv, mb * p.act);
  p.qk16 = after(p.qk16, mb * p.act);
  p.dout = after(p.dout, mb * p.act);
  if (p.out) p.out = after(p.out, mb * p.act);
  p.lse = after(p.lse, mb * p.act);
  p.delta = after(p.delta, mb * p.act);
  p.dqkv = after(p.dqkv, mb * p.grad);
  return p;
}

// Backward, key side.  A workgroup owns blocks of 32 keys, one or two waves each, and streams the
// query rows at and after them in tiles of 64: Q and dO, lse and delta, all by DMA.  Per wave and 32-query block:
//   S[q][k]  = Q K^T       (A = Q fragment from LDS, B = K fragment in registers)
//   dP[q][k] = dO V^T      (A = dO fragment from LDS, B = V fragment in registers)
//   P = exp(S/sqrt(D) - lse_q),  dS = P (dP - delta_q)
//   dV^T[d][k] += dO^T P   (A = transposing fragment of dO, B = P from the accumulator)
//   dK^T[d][k] += Q^T dS   (A = transposing fragment of Q,  B = dS)
// so a lane owns one key column and nothing moves between lanes.
// grid (heads, batch, key blocks): the key blocks with the most queries start first.
// F16S: the logits are recomputed from fp16 copies of Q and K (qk16, laid out like qkv) with
// the f16 instruction -- the operands the forward pass formed them from; everything else
// (V, dO, and Q and K as the operands of gradients) is bf16: the fp16 rows are a third tile.  Without F16S qk16 == qkv.
// RW x SW waves: RW blocks of 32 keys; with SW = 2 a second wave per block takes the other 32 queries
// of every tile and the two sums are added through LDS at the end.
template <bool F16S> constexpr int kBwdTiles = F16S ? 3 : 2;   // LDS tiles of a stage: [Q | dO | fp16 Q] or [K | V | fp16 K]
// The exponent is S/sqrt(D) - lse, rounded once, times log2(e), and delta is subtracted from the whole dP.  log2(e) taken into
// both terms beforehand, or dP begun at -delta, would be an operation an element less (1 % of both sides each at
// 1x8191x16x128), but round at the terms' size and not at the difference's: P's relative error at logits of 100, D = 64, 1.4e-7 ->
// 1.5e-6, at 32 and 128 9e-7 -> 2e-6.
template <int D, bool F16S, int RW, int SW>
__device__ __forceinline__ void dkv_block(const BwdArgs& args, int blk, char* lds, float (*stat)[2][BKV]) {
  const int mb = microbatch(args.B, args.act);
  const BwdArgs p = at_microbatch(args, mb);
  const bf16* const __restrict__ qkv = p.qkv;
  const bf16* const __restrict__ qk16 = p.qk16;
  const bf16* const __restrict__ dout = p.dout;
  const float* const __restrict__ lse = p.lse;
  const float* const __restrict__ delta = p.delta;
  bf16* const __restrict__ dqkv = p.dqkv;
  const int S = p.S, a = p.a;
  constexpr int KSTEPS = D / 16, DB = D / 32, TILE = BKV * D * 2, NW = RW * SW;
  const int lane = threadIdx.x & 63;
  const int lane_id = lane;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = blockIdx.x, b = blockIdx.y - mb * p.B;
  const int P = a * D;
  const size_t ld = 3 * (size_t)P;
  const bf16* base = qkv + (size_t)b * S * ld + (size_t)n * D;
  const bf16* base16 = qk16 + (size_t)b * S * ld + (size_t)n * D;
  const bf16* dobase = dout + (size_t)b * S * P + (size_t)n * D;
  const int ntile = (S + BKV - 1) / BKV;
  const float* lse_h = lse + ((size_t)b * a + n) * S;
  const float* delta_h = delta + ((size_t)b * a + n) * S;
  const int rw = wave % RW, half = wave / RW;
  const int k0 = blk * (32 * RW);
  const int kw0 = k0 + rw * 32;
  const int ql = lane & 31, h = lane >> 5;
  const int key = kw0 + ql;
  const int kclamp = key < S ? key : S - 1;
  const float rsd = 1.f / sqrtf((float)D);

  bf16x8 kfr[KSTEPS], vfr[KSTEPS];
#pragma unroll
  for (int kk = 0; kk < KSTEPS; ++kk) {
    kfr[kk] = *reinterpret_cast<const bf16x8*>(base16 + (size_t)kclamp * ld + P + kk * 16 + h * 8);
    vfr[kk] = *reinterpret_cast<const bf16x8*>(base + (size_t)kclamp * ld + 2 * P + kk * 16 + h * 8);
  }
#pragma unroll
  for (int kk = 0; kk < KSTEPS; ++kk) {
    settle(kfr[kk]);
    settle(vfr[kk]);
  }
  f32x16 dk[DB], dv[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) dk[i][e] = dv[i][e] = 0.f;

  const int aoff = natural_off<D>(ql, h);
  const int toff = tr_off<D>(lane);

  // The query tiles are walked from the LAST one down to the key block's own diagonal: every
  // key block of a head then starts at the same tile and they move in step, so the tiles one
  // workgroup streams are the ones its neighbours (same head, same XCD) are streaming at that
  // moment and come out of the L2 instead of HBM.  (Walking upwards from the diagonal, each
  // block is 256 rows ahead of the next one and the window does not fit the cache.)
  const int qt0 = k0 / BKV;
  auto fetch = [&](int qt, int stage) {
    // the lane index is made opaque here so that the per-lane DMA offsets are recomputed
    // (a dozen integer operations per tile) instead of being kept in registers across the
    // loop, where there are none to spare
    int lane = lane_id;
    asm volatile("" : "+v"(lane));
    char* t = lds + stage * kBwdTiles<F16S> * TILE;
    dma_tile<D, NW>(base, ld, qt * BKV, S, t, wave, lane);
    dma_tile<D, NW>(dobase, (size_t)P, qt * BKV, S, t + TILE, wave, lane);
    if constexpr (F16S) dma_tile<D, NW>(base16, ld, qt * BKV, S, t + 2 * TILE, wave, lane);
    const int qi = qt * BKV + lane;
    const int qc = qi < S ? qi : S - 1;
    if (wave == 0) dma_floats(lse_h, qc, stat[stage][0]);
    if (wave == 1) dma_floats(delta_h, qc, stat[stage][1]);
  };
  fetch(ntile - 1, 0);

  for (int qt = ntile - 1; qt >= qt0; --qt) {
    const int stage = (ntile - 1 - qt) & 1;
    asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    char* const tQ = lds + stage * kBwdTiles<F16S> * TILE;
    char* const tO = tQ + TILE;
    const char* const tQ16 = F16S ? tQ + 2 * TILE : tQ;
    if (qt > qt0) fetch(qt - 1, stage ^ 1);
    if ((qt + 1) * BKV > S) {   // (uniform) queries past the last one: p = ds = 0 has to meet zeros
      zero_rows<D, NW>(tQ, S - qt * BKV, wave, lane_id);
      zero_rows<D, NW>(tO, S - qt * BKV, wave, lane_id);
      __syncthreads();
    }
#pragma unroll 1
    for (int qb = SW == 2 ? half : 0; qb < (SW == 2 ? half + 1 : 2); ++qb) {
      const int qmin = qt * BKV + qb * 32;
      if (qmin + 31 < kw0 || qmin >= S) continue;  // block fully masked for this wave
      // S, then P = exp(S/sqrt(D) - lse) rounded to bf16 right away (the fp32 block dies
      // here: registers are the scarce resource of this kernel), then dP and
      // dS = P (dP - delta) with the rounded P -- the one that also enters dV.
      const float* Ls = &stat[stage][0][qb * 32 + h * 4];
      const float* Ds = &stat[stage][1][qb * 32 + h * 4];
      const bool masked = (qmin < kw0 + 31) || (qmin + 31 >= S);  // diagonal or ragged block
      bf16x8 pf[2], dsf[2];
      {
        f32x16 sacc;
#pragma unroll
        for (int e = 0; e < 16; ++e) sacc[e] = 0.f;
        GPTS_PRIO(1);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk)
          sacc = mma32<F16S>(natural_frag<D>(tQ16, aoff, qb, kk), kfr[kk], sacc);
        GPTS_PRIO(0);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 L = *reinterpret_cast<const f32x4*>(Ls + g * 8);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            sacc[g * 4 + e] = __builtin_amdgcn_exp2f(fmaf(sacc[g * 4 + e], rsd, -L[e]) * 1.4426950408889634f);
        }
        if (masked) {
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int query = qmin + (e >> 2) * 8 + h * 4 + (e & 3);
            if (key > query || query >= S) sacc[e] = 0.f;
          }
        }
        pf[0] = pack8(sacc, 0);
        pf[1] = pack8(sacc, 8);
        settle(pf[0]);
        settle(pf[1]);
      }
      {
        f32x16 dpacc;
#pragma unroll
        for (int e = 0; e < 16; ++e) dpacc[e] = 0.f;
        GPTS_PRIO(1);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk)
          dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(natural_frag<D>(tO, aoff, qb, kk), vfr[kk], dpacc, 0, 0, 0);
        GPTS_PRIO(0);
        if constexpr (D >= 64) {
          // dV's run of matrix instructions with dS between them, then dK's, instead of dS in front of both.  With dS from the
          // packed P, which leaves 16 conversions and 8 registers out, us for both sides, in front unpacked | in front from the
          // packed P | this: 1x8191x16x128 869 | 856 | 842, 1x2048x16x128 88.9 | 88.3 | 84.4, 4x1000x16x128 83.5 | 82.5 | 81.0,
          // 2x4096x32x64 517 | 506 | 497, 4x1024x16x64 50.3 | 48.4 | 46.9; no gain where a head has few blocks, 8x333x24x128 58.4 |
          // 59.5 | 58.7.  (The exponentials between dP's too: spills, 898 against 828 with dP begun at -delta at 1x8191x16x128; the
          // query side in such runs: 415 | 421 of its own.)
          constexpr int N = 2 * DB, AHEAD = 2;
          bf16x8 fr[2 * N];
          f32x4 Dl[4];
          auto load = [&](auto i_c) {
            constexpr int i = decltype(i_c)::value, x = i % N;
            fr[i] = tr_frag<D>(i < N ? tO : tQ, toff, qb * 2 + x / DB, x % DB);
          };
          // delta, four at a time, an instruction or two ahead of their elements; all in front where that has registers and other
          // workgroups hide it (D = 64 in one wave per 32 rows, 4x1024x16x64 47.6 -> 46.9; in two waves 4x8076x3x64 427 -> 470)
          constexpr bool IN_FRONT = D == 64 && SW == 1;
          auto load_delta = [&](int g) { Dl[g] = *reinterpret_cast<const f32x4*>(Ds + g * 8); };
          static_for<AHEAD>(load);
#pragma unroll
          for (int g = 0; g < (IN_FRONT ? 4 : 1); ++g) load_delta(g);
          __builtin_amdgcn_sched_barrier(0);
          static_for<2 * N>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value, x = i % N;
            // the elements of dS after instruction x: none after the first, beside which dP is completed
            constexpr int first = x < 2 ? 0 : (x - 1) * 16 / (N - 1), last = x * 16 / (N - 1);
            if constexpr (i + AHEAD < 2 * N) load(std::integral_constant<int, i + AHEAD>{});
            if constexpr (!IN_FRONT) {
#pragma unroll
              for (int g = 1; g < 4; ++g)
                if (i == 4 * g * (N - 1) / 16) load_delta(g);
            }
            if constexpr (i < N) {
              dv[x % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], pf[x / DB], dv[x % DB], 0, 0, 0);
#pragma unroll
              for (int e = first; e < last; ++e) dpacc[e] = element_of(pf, e) * (dpacc[e] - Dl[e >> 2][e & 3]);
              if constexpr (first < 8 && last >= 8) dsf[0] = pack8(dpacc, 0);
              if constexpr (last == 16) dsf[1] = pack8(dpacc, 8);
            } else {
              dk[x % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], dsf[x / DB], dk[x % DB], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
          });
          continue;
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 Dl = *reinterpret_cast<const f32x4*>(Ds + g * 8);
#pragma unroll
          for (int e = 0; e < 4; ++e) dpacc[g * 4 + e] = element_of(pf, g * 4 + e) * (dpacc[g * 4 + e] - Dl[e]);
        }
        dsf[0] = pack8(dpacc, 0);
        dsf[1] = pack8(dpacc, 8);
      }
      GPTS_PRIO(1);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {   // 16 queries per step
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          dv[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_frag<D>(tO, toff, qb * 2 + ks, db), pf[ks], dv[db], 0, 0, 0);
          dk[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_frag<D>(tQ, toff, qb * 2 + ks, db), dsf[ks], dk[db], 0, 0, 0);
        }
      }
      GPTS_PRIO(0);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  const float scale = 1.f / sqrtf((float)D);
  bf16* drow = dqkv + ((size_t)b * S + key) * ld + (size_t)n * D;
  if constexpr (SW == 2) {
    // the first wave of a key block finishes dK, the second dV: each hands the other its share, 32 columns at a time
    int at;   // the lane, found again: kept through the loop it was a register too many at D = 128
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(at));
    f32x4* ex = reinterpret_cast<f32x4*>(lds) + rw * (2 * 4 * kWave) + at;
    auto finish = [&](f32x16(&keep)[DB], f32x16(&give)[DB], int mine, float sc, size_t off) {
#pragma unroll
      for (int i = 0; i < DB; ++i) {
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 4; ++g)
          ex[((1 - mine) * 4 + g) * kWave] = f32x4{give[i][g * 4], give[i][g * 4 + 1], give[i][g * 4 + 2], give[i][g * 4 + 3]};
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 other = ex[(mine * 4 + g) * kWave];
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16)((keep[i][g * 4 + e] + other[e]) * sc);
          if (key < S) *reinterpret_cast<bf16x4*>(drow + off + i * 32 + g * 8 + h * 4) = o;
        }
      }
    };
    if (half == 0) finish(dk, dv, 0, scale, P);
    else finish(dv, dk, 1, 1.f, 2 * (size_t)P);
    return;
  }
  if (key < S) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 ok, ov;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ok[e] = (bf16)(dk[db][g * 4 + e] * scale);
          ov[e] = (bf16)dv[db][g * 4 + e];
        }
        *reinterpret_cast<bf16x4*>(drow + P + db * 32 + g * 8 + h * 4) = ok;
        *reinterpret_cast<bf16x4*>(drow + 2 * P + db * 32 + g * 8 + h * 4) = ov;
      }
  }
}

// Backward, query side.  A workgroup owns blocks of 32 queries and walks the key
// tiles of 64 up to the diagonal, everything transposed:
//   S^T = K Q^T,  dP^T = V dO^T  (A = K / V fragments from LDS, B = Q / dO in registers)
//   dS^T = P^T (dP^T - delta_q),  dQ^T[d][q] += K^T dS^T (A = transposing fragment of K).
// grid (heads, batch, query blocks), heaviest first.
// RW x SW waves as above, SW = 2 splitting the keys of a tile.
// out (may be null): the forward output (fp16 with F16S); delta_q = sum_d dO * O is then formed here, where dO is in
// registers anyway, and written for the key side, which runs after.  Null: delta is there already.
template <int D, bool F16S, int RW, int SW>
__device__ __forceinline__ void dq_block(const BwdArgs& args, int qt, char* lds) {
  const int mb = microbatch(args.B, args.act);
  const BwdArgs p = at_microbatch(args, mb);
  const bf16* const __restrict__ qkv = p.qkv;
  const bf16* const __restrict__ qk16 = p.qk16;
  const bf16* const __restrict__ dout = p.dout;
  const bf16* const __restrict__ out = p.out;
  const float* const __restrict__ lse = p.lse;
  float* const __restrict__ delta = p.delta;
  bf16* const __restrict__ dqkv = p.dqkv;
  const int S = p.S, a = p.a;
  constexpr int KSTEPS = D / 16, DB = D / 32, TILE = BKV * D * 2, NW = RW * SW, BW = 32 * RW, NKB = 2 / SW;
  const int lane = threadIdx.x & 63;
  const int lane_id = lane;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rw = wave % RW, kb0 = wave / RW * NKB;   // this wave's query block; its first key block of a tile
  const int n = blockIdx.x, b = blockIdx.y - mb * p.B;
  const int P = a * D;
  const size_t ld = 3 * (size_t)P;
  const bf16* base = qkv + (size_t)b * S * ld + (size_t)n * D;
  const bf16* base16 = qk16 + (size_t)b * S * ld + (size_t)n * D;
  const int q0 = qt * BW;
  const int ql = lane & 31, h = lane >> 5;
  const int qrow = q0 + rw * 32 + ql;
  const int qclamp = qrow < S ? qrow : S - 1;
  const int qmax_wave = min(q0 + rw * 32 + 31, S - 1);
  const float c = 1.4426950408889634f / sqrtf((float)D);

  bf16x8 qf[KSTEPS], dof[KSTEPS];
#pragma unroll
  for (int kk = 0; kk < KSTEPS; ++kk) {
    qf[kk] = *reinterpret_cast<const bf16x8*>(base16 + (size_t)qclamp * ld + kk * 16 + h * 8);
    dof[kk] = *reinterpret_cast<const bf16x8*>(dout + ((size_t)b * S + qclamp) * P + (size_t)n * D + kk * 16 + h * 8);
  }
  const float L2 = lse[((size_t)b * a + n) * S + qclamp] * 1.4426950408889634f;
  float Dl = 0.f;
  if (out) {   // (summed in attn_delta_kernel's order: a row's gradients do not depend on the form)
    float part[KSTEPS];
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
      const bf16x8 o = *reinterpret_cast<const bf16x8*>(out + ((size_t)b * S + qclamp) * P + (size_t)n * D + kk * 16 + h * 8);
      part[kk] = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) part[kk] = fmaf(F16S ? (float)__builtin_bit_cast(f16x8, o)[e] : (float)o[e], (float)dof[kk][e], part[kk]);
    }
#pragma unroll
    for (int x = KSTEPS / 2; x > 0; x >>= 1)
#pragma unroll
      for (int kk = 0; kk < x; ++kk) part[kk] += part[kk + x];
    Dl = part[0] + __shfl_xor(part[0], 32, 64);
    if (kb0 == 0 && h == 0 && qrow < S) delta[((size_t)b * a + n) * S + qrow] = Dl;
  } else {
    Dl = delta[((size_t)b * a + n) * S + qclamp];
  }
#pragma unroll
  for (int kk = 0; kk < KSTEPS; ++kk) {
    settle(qf[kk]);
    settle(dof[kk]);
  }
  settle(L2);
  settle(Dl);
  f32x16 dq[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) dq[i][e] = 0.f;

  const int koff = natural_off<D>(ql, h);
  const int toff = tr_off<D>(lane);

  const int last_key = min(q0 + BW, S);
  const int nkv = (last_key + BKV - 1) / BKV;
  auto fetch = [&](int kt, int stage) {
    int lane = lane_id;  // opaque: recompute the DMA offsets per tile rather than keep them
    asm volatile("" : "+v"(lane));
    char* t = lds + stage * kBwdTiles<F16S> * TILE;
    dma_tile<D, NW>(base + P, ld, kt * BKV, S, t, wave, lane);
    dma_tile<D, NW>(base + 2 * P, ld, kt * BKV, S, t + TILE, wave, lane);
    if constexpr (F16S) dma_tile<D, NW>(base16 + P, ld, kt * BKV, S, t + 2 * TILE, wave, lane);
  };
  fetch(0, 0);

  for (int kt = 0; kt < nkv; ++kt) {
    asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const int k0 = kt * BKV;
    char* const tK = lds + (kt & 1) * kBwdTiles<F16S> * TILE;
    const char* const tV = tK + TILE;
    const char* const tK16 = F16S ? tK + 2 * TILE : tK;
    if (kt + 1 < nkv) fetch(kt + 1, (kt + 1) & 1);
    if (k0 + BKV > S) {   // (uniform) keys past the last one: ds = 0 has to meet zeros
      zero_rows<D, NW>(tK, S - k0, wave, lane_id);
      __syncthreads();
    }
    const int kw0 = k0 + kb0 * 32;
    if (kw0 > qmax_wave) continue;
    f32x16 sacc[NKB], dpacc[NKB];
    GPTS_PRIO(1);
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
      for (int e = 0; e < 16; ++e) sacc[kb][e] = dpacc[kb][e] = 0.f;
#pragma unroll
      for (int kk = 0; kk < KSTEPS; ++kk) {
        sacc[kb] = mma32<F16S>(natural_frag<D>(tK16, koff, kb0 + kb, kk), qf[kk], sacc[kb]);
        dpacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(natural_frag<D>(tV, koff, kb0 + kb, kk), dof[kk], dpacc[kb], 0, 0, 0);
      }
    }
    GPTS_PRIO(0);
    if (kw0 + NKB * 32 - 1 > q0 + rw * 32) {  // tile reaches past the first query of the wave: mask
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          float p = __builtin_amdgcn_exp2f(fmaf(sacc[kb][e], c, -L2));
          const int key = kw0 + kb * 32 + (e >> 2) * 8 + h * 4 + (e & 3);
          if (key > qrow) p = 0.f;
          dpacc[kb][e] = p * (dpacc[kb][e] - Dl);
        }
    } else {
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float p = __builtin_amdgcn_exp2f(fmaf(sacc[kb][e], c, -L2));
          dpacc[kb][e] = p * (dpacc[kb][e] - Dl);
        }
    }
    GPTS_PRIO(1);
#pragma unroll
    for (int ks = 0; ks < 2 * NKB; ++ks) {
      const bf16x8 dsf = pack8(dpacc[ks >> 1], (ks & 1) * 8);
#pragma unroll
      for (int db = 0; db < DB; ++db)
        dq[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_frag<D>(tK, toff, kb0 * 2 + ks, db), dsf, dq[db], 0, 0, 0);
    }
    GPTS_PRIO(0);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  if constexpr (SW == 2) {
    __syncthreads();
    f32x4* ex = reinterpret_cast<f32x4*>(lds) + rw * (DB * 4 * kWave) + lane;
    if (kb0 != 0) {
#pragma unroll
      for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) ex[(i * 4 + g) * kWave] = f32x4{dq[i][g * 4], dq[i][g * 4 + 1], dq[i][g * 4 + 2], dq[i][g * 4 + 3]};
    }
    __syncthreads();
    if (kb0 != 0) return;
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 other = ex[(i * 4 + g) * kWave];
#pragma unroll
        for (int e = 0; e < 4; ++e) dq[i][g * 4 + e] += other[e];
      }
  }
  if (qrow < S) {
    const float scale = 1.f / sqrtf((float)D);
    bf16* drow = dqkv + ((size_t)b * S + qrow) * ld + (size_t)n * D;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (bf16)(dq[db][g * 4 + e] * scale);
        *reinterpret_cast<bf16x4*>(drow + db * 32 + g * 8 + h * 4) = o;
      }
  }
}

// Key side and query side a launch each, 32 RW rows per workgroup, the query side first (it forms delta): the form for
// many workgroups.  Held to 256 registers (they need 256 and 253 at head dimension 128, nothing spilt), two workgroups of four
// waves share a unit; left to itself the compiler took 278 and 304, and accumulators apart from the others.  Both sides,
// us: 2x4096x24x128 1005 | 687, 4x2048x24x128 562 | 389, 16x512x24x128 239 | 181, 2x4096x32x64 543 | 496, 1x8191x32x32 730 | 595.
template <int D, bool F16S, int RW> __global__ __launch_bounds__(64 * RW, 2) void attn_bwd_dkv_mfma_kernel(const BwdArgs p) {
  __shared__ __attribute__((aligned(1024))) char lds[2 * kBwdTiles<F16S> * BKV * D * 2];
  __shared__ __attribute__((aligned(256))) float stat[2][2][BKV];  // [stage][lse | delta][row]
  dkv_block<D, F16S, RW, 1>(p, blockIdx.z, lds, stat);
}
template <int D, bool F16S, int RW> __global__ __launch_bounds__(64 * RW, 2) void attn_bwd_dq_mfma_kernel(const BwdArgs p) {
  __shared__ __attribute__((aligned(1024))) char lds[2 * kBwdTiles<F16S> * BKV * D * 2];
  dq_block<D, F16S, RW, 1>(p, gridDim.z - 1 - blockIdx.z, lds);
}
// Both sides in one launch, 32 RW rows per workgroup, SW waves per block of 32: the forms for fewer
// workgroups.  Even z: key block z/2; odd z: the query blocks from the last one down (heaviest first).
// Two workgroups of four waves share a unit (not those of fp16 logits at D = 128, whose third tile leaves no room).
template <int D, bool F16S, int RW, int SW>
__global__ __launch_bounds__(64 * RW * SW, F16S && D == 128 && RW * SW == 4 ? 1 : 2) void attn_bwd_both_mfma_kernel(const BwdArgs p) {
  constexpr int TILES = 2 * kBwdTiles<F16S> * BKV * D * 2, EXCHANGE = SW == 2 ? RW * 2 * 4 * kWave * 16 : 0;
  __shared__ __attribute__((aligned(1024))) char lds[TILES > EXCHANGE ? TILES : EXCHANGE];
  __shared__ __attribute__((aligned(256))) float stat[2][2][BKV];
  const int i = blockIdx.z >> 1;
  if ((blockIdx.z & 1) == 0)
    dkv_block<D, F16S, RW, SW>(p, i, lds, stat);
  else
    dq_block<D, F16S, RW, SW>(p, (int)(gridDim.z >> 1) - 1 - i, lds);
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// How the rows go over the workgroups.  A workgroup walks its rows' half of the other side tile by
// tile, so with few workgroups the time is that chain; fewer rows per workgroup and two waves per 32
// rows, which share a tile, shorten it, at the price of streaming each tile for fewer rows.  The price
// shows as soon as the workgroups no longer run at once, and a short sequence has no long chain to
// shorten: the limits, in blocks of 64 rows (n), grow with S and are lower where a tile is more bytes.
// Measured at the lines in us, both sides:
//   forward, 128 rows and one wave per 32 | 64 rows and two waves:
//      D=128  S=128   n 256   7.0 |  6.5    n 320   7.3 |  8.4      S=512   n 512  15.8 | 14.4    n 640  18.1 | 17.6
//             S=1024  n 768  29.7 | 27.3    n1024  31.3 | 33.7      S=4096  n1024 102.3 | 96.8    n1280   112 |  118
//      D=64   S=256   n 640   8.0 |  7.8    n 768   8.2 |  8.7      S=1024  n1024  19.9 | 19.4    n1280  22.2 | 24.2
//             S=4096  n1280  71.0 | 67.4    n1536  76.0 | 78.2
//      D=32   S=256   n 768   5.8 |  6.0    n 896   5.9 |  6.3      S=1024  n1152  16.0 | 15.6    n1280  15.6 | 16.7
//             S=4096  n1280  49.1 | 48.2    n1536  53.7 | 55.5
//   forward, time of 256 rows and eight waves, which copy each tile for twice the rows, over that of 128 rows and four waves,
//      D=128, bf16 and fp16 alike: whole pairs of rounds of the compute units or just under, the last workgroup of a sequence
//      more than half full, one pair: S 1000 ... 1500 0.94 ... 1.06, beyond 0.92 ... 1.00 (4x2048x16 0.98, 1x4096x32 0.97, 1x8191x16
//      0.94); more pairs: S 1000 ... 1700 0.93 ... 1.08 and 16x1024x16 1.19, ... 2200 0.93 ... 1.04, beyond 0.95 ... 1.01 (2x4096x32
//      0.98); the last at most half full: S 1000 ... 2000 1.03 ... 1.14, ... 5000 1.00 ... 1.10, beyond 5900 0.97 ... 0.99.  Not just
//      under pairs: 1x6000x16 1.05, 4x1024x40 1.08, 1x4096x24 1.07, 2x1984x16 1.09.
//   backward, 128 rows and one wave per 32, one launch | 64 rows and two waves, one launch:
//      D=128  S=128   n 128  13.9 | 12.9    n 192  14.7 | 16.4      S=256   n 256  21.4 | 19.9    n 320  24.0 | 24.6
//             S=512   n 448  36.9 | 36.8    n 512  38.0 | 39.2      S=1024  n 576  63.3 | 61.6    n 640  64.5 | 67.7
//             S=2048  n 640   114 |  107    n 768   118 |  123      S=4096  n 768   223 |  222    n 896   234 |  249
//      D=64   S=128   n 128   9.9 |  9.0    n 192  10.3 | 10.5      S=256   n 384  16.2 | 15.0    n 448  16.6 | 18.0
//             S=512   n 576  25.7 | 24.8    n 640  26.2 | 26.5      S=1024  n 896  45.6 | 46.5    n1152  57.6 | 58.0
//             S=2048  n1024  83.1 | 82.9    n1280   105 |  104      S=4096  n1536   222 |  220    n1792   254 |  255
//      D=32   S=128   n 384   9.1 |  8.9    n 448   9.3 |  9.6      S=256   n 512  12.3 | 12.1    n 576  13.6 | 13.6
//             S=512   n 768  21.2 | 19.8    n 896  22.0 | 22.2      S=1024  n1024  34.6 | 33.2    n1152  35.7 | 37.0
//             S=4096  n1536   148 |  143    n1792   166 |  166
//   backward, time of a launch each over that of one launch of 128 rows (which needs delta from a pass of its own, and whose two
//      kinds of workgroup share no tiles), S 192 ... 16384, D=128 | 64 | 32: n 1280 0.97 ... 1.13 | 1.00 ... 1.08 | 1.05 ... 1.26, n 1536
//      0.98 ... 1.05 | 0.95 ... 1.03 | 1.04 ... 1.11, n 1792 0.97 ... 1.07 | 0.96 ... 1.01 | 1.04 ... 1.10, n 2048 0.91 ... 1.03 |
//      0.92 ... 0.98 | 0.95 ... 1.05.
//   backward, a launch each, time of 256 rows over 128: D=128, S >= 3500, whole pairs of rounds of the compute units or
//      just under: n 2048 0.93, n 4096 0.96; between: n 3072 1.00; S=2048 n 2048 0.97, n 3072 1.01; S=1024 n 3072 1.04; S=512
//      1.09; D=64 and 32 1.0 ... 1.3 everywhere.
// (192 rows are three blocks of 64 or two of 128, whose second one is half empty: a limit of their own at D=32.)
long row_blocks(int B, int S, int a, int rows) { return (long)a * B * ((S + rows - 1) / rows); }
struct Limit { int rows, most; };   // sequences of up to `rows`: at most so many blocks of 64 rows
template <int N> bool within(const Limit (&t)[N], int B, int S, int a) {
  int i = 0;
  while (i < N - 1 && S > t[i].rows) ++i;
  return row_blocks(B, S, a, 64) <= t[i].most;
}
constexpr int kAnyRows = 0x7fffffff;
bool split_fwd(int B, int S, int a, int d) {
  static constexpr Limit k128[] = {{64, 0},     {192, 256},  {320, 480},  {512, 576},  {1023, 704},
                                   {1535, 768}, {2047, 816}, {4095, 928}, {kAnyRows, 1024}};
  static constexpr Limit k64[] = {{64, 0}, {192, 480}, {320, 640}, {640, 768}, {1499, 1024}, {4095, 1152}, {kAnyRows, 1280}};
  static constexpr Limit k32[] = {{64, 1280}, {128, 768}, {192, 1536}, {400, 768}, {699, 912}, {4095, 1152}, {kAnyRows, 1280}};
  return d == 128 ? within(k128, B, S, a) : d == 64 ? within(k64, B, S, a) : within(k32, B, S, a);
}
// workgroups of 256 rows in whole pairs of rounds, a heavy one and a light one, or just under
bool pairs_of_rounds(int B, int S, int a) {
  const long wg = row_blocks(B, S, a, 256), pairs = (wg + 511) / 512;
  return 7 * (pairs * 512 - wg) <= 512;
}
// such workgroups for the forward: the last one of a sequence more than half full, unless it is one of many
bool eight_waves_fwd(int B, int S, int a) {
  if (!pairs_of_rounds(B, S, a)) return false;
  if ((S - 1) % 256 < 128) return S >= 5500;
  return S >= (row_blocks(B, S, a, 256) <= 512 ? 1500 : 2200);
}
enum BwdForm { BWD_SPLIT64, BWD_BOTH128, BWD_EACH128, BWD_EACH256 };
BwdForm bwd_form(int B, int S, int a, int d) {
  static constexpr Limit k128[] = {{64, 0},     {128, 128},  {192, 256},  {320, 288},       {512, 448},
                                   {700, 512}, {1200, 576}, {2999, 640}, {kAnyRows, 768}};
  static constexpr Limit k64[] = {{64, 0},     {128, 128},  {192, 256},   {320, 384},       {512, 576},
                                  {800, 640}, {1500, 896}, {2999, 1024}, {kAnyRows, 1536}};
  static constexpr Limit k32[] = {{64, 0},     {128, 384},   {256, 512},   {400, 640},
                                  {800, 768}, {1500, 1024}, {3500, 1152}, {kAnyRows, 1536}};
  if (d == 128 ? within(k128, B, S, a) : d == 64 ? within(k64, B, S, a) : within(k32, B, S, a)) return BWD_SPLIT64;
  if (row_blocks(B, S, a, 64) <= 1700) return BWD_BOTH128;
  return d == 128 && pairs_of_rounds(B, S, a) && (S >= 3500 || row_blocks(B, S, a, 256) <= 512) ? BWD_EACH256 : BWD_EACH128;
}

template <int D, bool F16>
void launch_fwd(const bf16* qkv, bf16* out, float* lse, int B, int S, int a, int n, size_t stride, hipStream_t st) {
  auto grid = [&](int rows) { return dim3(a, B * n, (S + rows - 1) / rows); };
  if (split_fwd(B, S, a, D)) {
    hipLaunchKernelGGL((attn_fwd_mfma_kernel<D, F16, 2, 2>), grid(64), dim3(256), 0, st, qkv, out, lse, S, a, B, stride);
    return;
  }
  if constexpr (D == 128) {
    if (eight_waves_fwd(B, S, a)) {
      hipLaunchKernelGGL((attn_fwd_mfma_kernel<D, F16, 8, 1>), grid(256), dim3(512), 0, st, qkv, out, lse, S, a, B, stride);
      return;
    }
  }
  hipLaunchKernelGGL((attn_fwd_mfma_kernel<D, F16, 4, 1>), grid(128), dim3(256), 0, st, qkv, out, lse, S, a, B, stride);
}

template <int D, bool F16> void launch_bwd(const bf16* out, BwdArgs p, int n, hipStream_t st) {
  const int B = p.B;
  auto grid = [&](int rows, int sides) { return dim3(p.a, B * n, sides * ((p.S + rows - 1) / rows)); };
  auto both = [&](auto rw_c, auto sw_c) {   // delta beforehand
    constexpr int RW = decltype(rw_c)::value, SW = decltype(sw_c)::value;
    const int total = B * p.S * p.a;
    hipLaunchKernelGGL((attn_delta_kernel<D, F16>), dim3((total + 2048 / D - 1) / (2048 / D), n), dim3(256), 0, st, out, p.dout, p.delta, p.S, p.a, total, p.act);
    hipLaunchKernelGGL((attn_bwd_both_mfma_kernel<D, F16, RW, SW>), grid(32 * RW, 2), dim3(64 * RW * SW), 0, st, p);
  };
  auto each = [&](auto rw_c) {
    constexpr int RW = decltype(rw_c)::value;
    p.out = out;
    hipLaunchKernelGGL((attn_bwd_dq_mfma_kernel<D, F16, RW>), grid(32 * RW, 1), dim3(64 * RW), 0, st, p);
    hipLaunchKernelGGL((attn_bwd_dkv_mfma_kernel<D, F16, RW>), grid(32 * RW, 1), dim3(64 * RW), 0, st, p);
  };
  using std::integral_constant;
  const BwdForm form = bwd_form(B, p.S, p.a, D);
  if constexpr (F16 && D == 128) {   // one workgroup per unit: eight waves
    if (form == BWD_SPLIT64 || form == BWD_BOTH128) both(integral_constant<int, 4>{}, integral_constant<int, 2>{});
    else each(integral_constant<int, 8>{});
  } else {
    if (form == BWD_SPLIT64) return both(integral_constant<int, 2>{}, integral_constant<int, 2>{});
    if (form == BWD_BOTH128) return both(integral_constant<int, 4>{}, integral_constant<int, 1>{});
    if constexpr (D == 128) {
      if (form == BWD_EACH256) return each(integral_constant<int, 8>{});
    }
    each(integral_constant<int, 4>{});
  }
}

}  // namespace

// The kernels address a tile row with a 32-bit byte offset from the (batch, head) base and
// count (batch, row, head) triples in an int.
bool attention_mfma_supported(int B, int S, int a, int d) {
  return (d == 32 || d == 64 || d == 128) && B >= 1 && S >= 1 && a >= 1 && (size_t)S * 3 * a * d < (1ull << 31) &&
         (size_t)B * S * a < (1ull << 27);
}

// (the sequences of a single call are left to the launch, which takes 65536 of them)
static bool microbatches_fit(int B, int n) { return n == 1 || (n > 1 && (long)B * n <= 65535); }

size_t attention_mfma_scratch_bytes(int B, int S, int a, int d, int phase) {
  // forward uses none; the least amount keeps a null scratch refused, as where it does
  return phase == 0 ? 256 : align256((size_t)B * a * S * sizeof(float));   // delta
}

hipError_t attention_fwd_mfma(int B, int S, int a, int d, const void* qkv, void* out, float* lse,
                              hipStream_t st, bool f16, int n, size_t stride) {
  if (!attention_mfma_supported(B, S, a, d) || !microbatches_fit(B, n)) return hipErrorInvalidValue;
  const bf16* q = (const bf16*)qkv;
#define GPTS_FWD(D)                                                    \
  do {                                                                 \
    if (f16) launch_fwd<D, true>(q, (bf16*)out, lse, B, S, a, n, stride, st);     \
    else launch_fwd<D, false>(q, (bf16*)out, lse, B, S, a, n, stride, st);        \
  } while (0)
  if (d == 128) GPTS_FWD(128);
  else if (d == 64) GPTS_FWD(64);
  else GPTS_FWD(32);
#undef GPTS_FWD
  return hipGetLastError();
}

hipError_t attention_bwd_mfma(int B, int S, int a, int d, const void* qkv, const void* out,
                              const float* lse, const void* dout, void* dqkv, void* scratch,
                              hipStream_t st, const void* qkv_f16, int n, size_t act, size_t grad) {
  if (!attention_mfma_supported(B, S, a, d) || !microbatches_fit(B, n)) return hipErrorInvalidValue;
  const bf16* q = (const bf16*)qkv;
  const bf16* o = (const bf16*)out;
  const bool f16 = qkv_f16 != nullptr;
  const BwdArgs p{q, f16 ? (const bf16*)qkv_f16 : q, (const bf16*)dout, nullptr, lse, static_cast<float*>(scratch), (bf16*)dqkv, S, a, B, act, grad};
#define GPTS_BWD(D)                             \
  do {                                          \
    if (f16) launch_bwd<D, true>(o, p, n, st);  \
    else launch_bwd<D, false>(o, p, n, st);     \
  } while (0)
  if (d == 128) GPTS_BWD(128);
  else if (d == 64) GPTS_BWD(64);
  else GPTS_BWD(32);
#undef GPTS_BWD
  return hipGetLastError();
}

}  // namespace gpts

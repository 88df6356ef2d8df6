// The bf16 (and, for the forward phase of cfg.fwd_fp16 stages, fp16) matrix-product kernel of
// gfx950, fp32 accumulation, for the three forms the stage needs:
//   NT  C[M,N]   = A[M,K] B[N,K]^T     forward linears   (both operands K-contiguous)
//   NN  C[M,N]   = A[M,K] B[K,N]       data gradients    (B is K-major)
//   TN  Cf[M,N] += A[K,M]^T B[K,N]     weight gradients  (both operands K-major)
// gemm_mfma.hip chooses the tile; gemm_fwd*.hip, gemm_dgrad.hip and gemm_wgrad.hip hold the instances.
//
// One workgroup: 2 x 2 waves, a 32 MB x 32 NB tile, K in slices of BK through a ring of NS LDS stages,
// v_mfma_f32_16x16x32 with the wave's MB x NB accumulator blocks of 16 x 16 placed by hand in AGPRs:
// block (ib, jb) lives in a[4(NB ib + jb) .. +3] for the whole kernel, the matrix instructions are
// inline assembly naming those registers (agpr_ops.hpp) and the epilogue reads them with
// v_accvgpr_read.  (The compiler moves that many small accumulators between the register files in
// every iteration; the chip sustains a higher clock on 16x16x32 than on the same flops as
// 32x32x16: 2.05 against 1.80 GHz on matrix instructions alone.)
// What bounds it: the clock the matrix pipe's power leaves (about 1400 TFLOP/s of random bf16) where
// the tiles fill the chip, the latency of the copies below that.  Loaded, a slice takes about 2 us
// to arrive, so what counts is how many bytes are in flight: slices of 64 k (whole 128-byte lines of
// a K-contiguous row, half the barriers) and as many stages as fit 160 KB.  4096x1024x4096, 256 tiles
// of 128x128: two stages of 64 (64 KB) 44 us, three or four 30 us; 2048x5120x5120, 256 tiles of
// 256x160: slices of 32, four stages (104 KB) 100 us, slices of 64, three stages (156 KB) 78 us.
//  * Slices go global -> LDS by the DMA path (global_load_lds_dwordx4: no registers, no ds_write),
//    issued from inline assembly and waited for with explicit vmcnt counts, spread between the
//    matrix instructions: a wave blocked on issuing a DMA cannot issue MFMAs, and the compiler
//    would drain every DMA (vmcnt(0)) in front of every transposing LDS read.
//  * Fragments are double buffered in registers: while one k = 32 step is multiplied the
//    fragments of the next are read from LDS, so a stage is free for the slice NS ahead as soon as
//    its last step begins.  One barrier per slice, in front of that step.
//  * The DMA writes 16-byte slots in lane order, so bank-conflict avoidance is done by choosing
//    WHICH global chunk a lane fetches (an XOR swizzle of the chunk index), never by padding.
//    Weight images (prepare_image_kernel) store a weight in exactly that LDS order, so that every
//    DMA instruction copies 1 KiB of contiguous memory.
//  * K-major operands are stored in LDS as they sit in memory ([k][rows]) and fragments are read
//    with the transposing LDS load ds_read_b64_tr_b16, so no operand is ever transposed in HBM.
//  * The two MFMA operands are swapped (D = B-fragment x A-fragment): lane l holds, for output row
//    l % 16 of a block, the four columns 4 (l / 16) .. +3.  The epilogue stages the wave's block
//    through the (then free) pipeline LDS and reads it back row-major, so that every global access
//    of the fused bias / GeLU / GeLU' / residual / fp32-accumulate epilogues covers whole lines.
//  * Workgroup -> tile map: consecutive workgroup ids land on different XCDs, so ids are first
//    regrouped per XCD and then walked in bands of 4 tile rows to keep each XCD's L2 working
//    set to a compact patch of the output.
#pragma once
#include <type_traits>
#include <utility>

#include "agpr_ops.hpp"
#include "reduce.hpp"

namespace gpts {

// epilogue kinds
// (RES32: the residual is fp32; OUT32: C is written as fp32 -- the residual stream of a bf16 stage)
enum { EPI_BIAS_RES = 0, EPI_GELU_TANH, EPI_GELU_ERF, EPI_PLAIN, EPI_DGELU_TANH, EPI_DGELU_ERF, EPI_ACCUM,
       EPI_BIAS_RES32_OUT32, EPI_BIAS_RES32_OUT16, EPI_BIAS /* bias only: no residual operand */,
       EPI_ONCE = 16 /* added to a kind: see MfmaArgs::once */ };

struct MfmaArgs {
  const bf16* A;
  const bf16* B;
  void* C;
  int M, N, K;
  const bf16* bias;
  const void* residual;
  bf16* gelu_out;
  const bf16* dgelu_u;
  float* colsum;   // GeLU' epilogue only, may be null: column sums of C per group of tile rows
  // The accumulated matrix, or the pre-activation u that a GeLU epilogue writes and a GeLU' epilogue reads, goes past the
  // caches non-temporally and pushes no operand out of them.  It is met again only after more has passed than they hold, but
  // for u where a backward pass recomputes, which reads it once more right behind; measured with kOnceBytes.
  int once = 0;
  int b_img = 0;   // B is the weight's tiled image (tiles of 256 rows, slices of kImageK): kernels with BK = kImageK only
  // The tokens of several micro-batches, each in its own buffer.
  // K-major products (weight gradients): the contraction runs over `batch` pieces of
  // K rows each (K is then the length of ONE piece), piece s of A starting stride_a elements
  // after piece s-1, likewise B and stride_b.
  // The others: `batch` products with the same B, whose tile rows follow on, the next A, C, residual or dgelu_u
  // stride_a, stride_b, 16 stride_r bytes on (see GemmEpilogue).
  int batch = 1;
  uint32_t stride_r = 0;
  size_t stride_a = 0, stride_b = 0;
};

constexpr int kImageK = 64;   // slice depth of the weight images

// The tiles there are instances of, largest first.
enum Tile { TILE_256x256 = 0, TILE_256x192, TILE_256x160, TILE_192x192, TILE_256x128, TILE_128x128, TILE_128x64,
            TILE_64x64, TILE_64x32, N_TILES };

// Forward products and data gradients in more than one tile of 128x128 or 128x64 per compute unit: two stages, so
// that two (three) workgroups share a unit and one's stores run under the other's slices.  With four stages a
// unit holds one, which waits for its first slice and its stores in every round.  Four | two stages, us: GeLU'
// 7784x9152, K = 256, 128x128 143 | 101; bias 9920x15872, K = 64 156 | 90; GeLU 8192x3072, K = 768 75 | 55; GeLU'
// 4096x4096, K = 1024 in 128x64 84 | 64, 128x128 58 | 45; bias 3968x2048, K = 2048 37 | 32.  Time of two over four
// stages, 288 to 1536 tiles: 128x128 K to 256 0.77, to 768 0.91, to 1536 0.82, to 3072 0.87; 128x64 K = 832 0.83, to 3072
// 0.92; with at most 256 tiles 0.99 ... 1.05 up to 768, 1.1 at 1024 to 1.5 beyond.
constexpr int kShortSlices = 12, kSharedSlices = 64;   // of 64 k
inline bool short_contraction(long K) { return (K + 63) / 64 <= kShortSlices; }
inline bool two_stages(long tiles, long K) { return tiles > 256 && (K + 63) / 64 <= kSharedSlices; }

// Launchers, one translation unit each.
hipError_t launch_gemm_fwd(Tile tile, int epi, const MfmaArgs& a, hipStream_t st);
hipError_t launch_gemm_fwd_f16(Tile tile, int epi, const MfmaArgs& a, hipStream_t st);
hipError_t launch_gemm_dgrad(Tile tile, int epi, const MfmaArgs& a, hipStream_t st);
// n <= kMaxWgrads products and n_sums <= kMaxReduceSegs partial sums, one launch
hipError_t launch_gemm_wgrad(Tile tile, const MfmaArgs* a, int n, const ReduceSeg* sums, int n_sums, hipStream_t st);

// 16-byte chunk swizzle of a K-contiguous tile row of eight chunks (BK = 64).  A 16-byte LDS read serves
// 16 lanes at a time over the 64 banks, lanes {0-3, 12-15, 20-27} of each half wave, then the others, and
// not 16 in a row: of a fragment (lane: row lane % 16, chunk lane / 16) rows 4-11 of the one chunk come
// together with rows 0-3 and 12-15 of the chunk before it.  The eighth bit of the row (its half of the 64 banks)
// and this make the 16 places different.
__host__ __device__ __forceinline__ int swz_kc(int row) { return (row & 7) ^ ((row >> 2) & 1); }

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));

// Per-lane state of one operand: global offsets for the DMA and LDS offsets for the fragment
// reads.  R = tile rows, BK = slice depth.
// K-contiguous: [R rows][BK], 16-byte chunks swizzled with the row.
// K-major: column panels of PW columns, each [BK k-rows][PW], 32-byte units swizzled with the
// k-row; PW is the whole tile where its width is a multiple of 128 (the swizzle then has eight
// units to spread over), else 64 or 32.
template <int R, int BK, bool KMAJOR> struct Operand {
  static constexpr int NW = 4;                        // waves that share the copying
  static constexpr int BYTES = R * BK * 2;
  static constexpr int NINST = BYTES / 1024;          // DMA instructions (1 KiB each) per slice
  static constexpr int NI = (NINST + NW - 1) / NW;    // per wave; the last wave may repeat the last one
  static constexpr int RB = BK * 2;                   // bytes per row of a K-contiguous tile
  static constexpr int CPR = BK / 8;                  // 16-byte chunks per such row
  static constexpr int PW = R % 128 == 0 ? R : (R % 64 == 0 ? 64 : 32);
  static constexpr int ROWB = PW * 2, PANEL = BK * ROWB;
  static_assert(BYTES % 1024 == 0, "whole DMA instructions");
  uint32_t goff[NI];                        // byte offset of this lane's chunk in slice 0

  static __device__ __forceinline__ int inst(int wave, int i) { return min(wave * NI + i, NINST - 1); }
  static __device__ __forceinline__ int swz_km(int k) {
    if constexpr (PW >= 128) return ((k & 3) << 1) | ((k >> 3) & 1);
    else if constexpr (PW == 64) return ((k >> 1) & 1) | (((k >> 3) & 1) << 1);
    else return (k >> 3) & 1;
  }
  // LDS offset of the 32-byte unit holding columns c0 .. c0+15 (c0 a multiple of 16) of k-row k
  static __device__ __forceinline__ int unit_off(int k, int c0) {
    return (c0 / PW) * PANEL + k * ROWB + ((((c0 % PW) >> 4) ^ swz_km(k)) << 5);
  }

  __device__ __forceinline__ void init(int r0, int rtotal, size_t ld, int wave, int lane, bool img) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int slot = inst(wave, i) * 64 + lane;
      if constexpr (!KMAJOR) {
        const int row = slot / CPR;
        if (img) {
          // image: [tile of 256 rows][slice][256 x BK]; the rows past the last image tile repeat its end
          const int rpad = (rtotal + 255) / 256 * 256;
          const int gr = min(r0 + row, rpad - 16 + (row & 15));
          goff[i] = (uint32_t)(((size_t)(gr / 256) * 256 * ld + (size_t)(gr % 256) * BK + (slot % CPR) * 8) * 2);
        } else {
          const int chunk = (slot % CPR) ^ swz_kc(row);
          const int gr = min(r0 + row, rtotal - 1);
          goff[i] = (uint32_t)(((size_t)gr * ld + chunk * 8) * 2);
        }
      } else {
        const int byte = slot * 16, panel = byte / PANEL, k = byte % PANEL / ROWB, wb = byte % ROWB;
        const int col = panel * PW + (((wb >> 5) ^ swz_km(k)) << 4) + ((wb >> 4) & 1) * 8;
        const int gc = (r0 + col < rtotal) ? r0 + col : 0;
        goff[i] = (uint32_t)(((size_t)k * ld + gc) * 2);
      }
    }
  }

  // Enqueue DMA instruction i (a compile-time constant after unrolling) of the slice at `base`:
  // 64 lanes x 16 bytes from base + goff -> 1 KiB of LDS (wave-uniform address, passed in M0).
  // Written as inline assembly on purpose: the compiler then does not track these copies, so it
  // neither drains them (vmcnt(0)) in front of LDS reads it cannot prove independent, nor counts
  // them; completion is waited for explicitly.
  __device__ __forceinline__ void issue(const bf16* __restrict__ base, uint32_t lds_tile, int wave, int i) const {
    const uint32_t dst = lds_tile + inst(wave, i) * 1024;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 ::"s"(dst), "v"(goff[i]), "s"(base)
                 : "memory");
  }
};

// eight bf16 from two transposing LDS reads (each delivers 4 consecutive k of the lane's column)
__device__ __forceinline__ bf16x8 tr_pair(const char* p0, const char* p1) {
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p0);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p1);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Wait until at most VM of this wave's DMA instructions are still in flight and all of its LDS
// reads have returned, then meet the other waves.  (A plain barrier intrinsic would make the
// compiler drain every outstanding DMA first.)
template <int VM> __device__ __forceinline__ void wait_dma_and_barrier() {
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::"n"(VM) : "memory");
}

template <int... I, class F> __device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>): a loop whose index is a constant expression
template <int N, class F> __device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// ---- epilogue --------------------------------------------------------------------
// A wave's staged rows: WN fp32 columns, 16-byte chunks XOR-swizzled with the row where their
// number is a power of two, else rows padded by 16 bytes: either way the eight lanes that write
// one column chunk of eight rows together hit different banks.
template <int WN> struct Staged {
  static constexpr int CW = WN / 4;
  static constexpr bool XOR = (CW & (CW - 1)) == 0;
  static constexpr int PITCH = XOR ? WN : WN + 4;   // floats
  static __device__ __forceinline__ int slot(int row, int chunk) {
    return row * PITCH + (XOR ? (chunk ^ (row & (CW - 1))) : chunk) * 4;
  }
};

// Accesses to what nobody reads again soon (MfmaArgs::once): non-temporal.
template <bool NT, typename V> __device__ __forceinline__ V load_once(const V* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, typename V> __device__ __forceinline__ void store_once(V* p, const V& v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// The accumulators hold a lane-per-row layout, which would store 16-byte pieces scattered over 16
// rows.  Each wave instead stages its rows through LDS in passes of RP rows (write_pass(pass)) and
// reads them back row-major: CW lanes cover one row of the WN columns, so every global load and
// store touches whole cache lines.
// OUT16: the 16-bit outputs (C of the bias-only epilogue; C and the GeLU output of the GeLU
// epilogues) are written as fp16 instead of bf16 (forward activations kept in fp16).
//
// What an epilogue reads that depends on addresses only (the bias, and the first batch of the fp32 tile that an
// accumulating product adds to, of a residual, of u for GeLU') is asked for by begin(): in tiles up to 128x64 in front of the
// slices (EARLY), so that no memory latency follows the last one, else after them.  After | in front, us a step: 192
// tokens 320 wide (64x32 and 64x64 tiles, five slices) 290.3 | 282.7; in 128x128, whose products are long enough to lose
// more by the later slices and the registers, 4096 tokens 1024 wide 1935 | 1950, backward of 2048 tokens 2048 wide 1207 | 1220.
template <int KIND, bool OUT16, int WM, int WN, int RP> struct GemmEpi {
  static constexpr int EPI = KIND & ~EPI_ONCE;
  static constexpr bool ONCE = (KIND & EPI_ONCE) != 0;
  static_assert(!OUT16 || EPI == EPI_BIAS || EPI == EPI_GELU_TANH || EPI == EPI_GELU_ERF ||
                    EPI == EPI_BIAS_RES32_OUT32 || EPI == EPI_BIAS_RES32_OUT16,
                "fp16 outputs exist for the forward epilogues only");
  static constexpr bool EARLY = WM * WN <= 64 * 32;
  static constexpr int CW = Staged<WN>::CW, RPI = 64 / CW;          // chunks per row, rows per read instruction
  static constexpr bool FULL = 64 % CW == 0;                        // no idle lanes
  static constexpr bool RES32 = EPI == EPI_BIAS_RES32_OUT32 || EPI == EPI_BIAS_RES32_OUT16;
  static constexpr bool GELU = EPI == EPI_GELU_TANH || EPI == EPI_GELU_ERF;
  static constexpr bool DGELU = EPI == EPI_DGELU_TANH || EPI == EPI_DGELU_ERF;
  static constexpr bool BIAS = EPI == EPI_BIAS_RES || EPI == EPI_BIAS || RES32 || GELU;
  // The readback goes in batches of UB row instructions.  The global loads of a batch are issued one batch ahead,
  // and a batch's memory latency overlaps the staging and the arithmetic and stores of the
  // batch before it.
  static constexpr int ITS = (RP + RPI - 1) / RPI, UB = ITS < 4 ? ITS : (ITS % 8 == 0 || ITS > 16 ? 8 : 4);
  static constexpr int NPASS = WM / RP, BPP = (ITS + UB - 1) / UB, NBATCH = NPASS * BPP;
  static constexpr bool EXACT = BPP * UB * RPI == RP && FULL;        // no row past the pass's last
  static_assert(WM % RP == 0, "whole passes");
  static constexpr bool HAS_LOADS = EPI == EPI_ACCUM || RES32 || DGELU || EPI == EPI_BIAS_RES;
  struct Batch {
    f32x4 in32[UB];
    bf16x4 in16[UB];
    bool ok[UB];
    size_t o[UB];
  };
  const MfmaArgs a;   // (a copy: by reference the arguments would live in memory)
  const int m_first, rd_chunk, rd_row, n;
  const bool n_ok;
  bf16x4 bias;
  Batch bt[2];

  // m_first, n_first: output row and column of the wave's first element; WM rows in all
  __device__ __forceinline__ GemmEpi(const MfmaArgs& a_, int m_first_, int n_first, int lane)
      : a(a_), m_first(m_first_), rd_chunk(lane % CW), rd_row(lane / CW), n(n_first + lane % CW * 4),
        n_ok(n_first + lane % CW * 4 < a_.N && (FULL || lane / CW < RPI)) {}

  template <int idx> __device__ __forceinline__ void issue() {
    constexpr int pass = idx / BPP, it0 = (idx % BPP) * UB;
    Batch& t = bt[idx & 1];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int row = (it0 + u) * RPI + rd_row;
      const int m = m_first + pass * RP + row;
      t.ok[u] = m < a.M && n_ok && (EXACT || row < RP);
      t.o[u] = t.ok[u] ? (size_t)m * a.N + n : 0;  // element 0 is always a valid address
      if constexpr (EPI == EPI_ACCUM) t.in32[u] = load_once<ONCE>(reinterpret_cast<const f32x4*>(static_cast<const float*>(a.C) + t.o[u]));
      if constexpr (RES32) t.in32[u] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.residual) + t.o[u]);
      if constexpr (DGELU) t.in16[u] = load_once<ONCE>(reinterpret_cast<const bf16x4*>(a.dgelu_u + t.o[u]));
      if constexpr (EPI == EPI_BIAS_RES) t.in16[u] = *reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(a.residual) + t.o[u]);
    }
  }
  __device__ __forceinline__ void begin() {
    if constexpr (BIAS) {
#pragma unroll
      for (int e = 0; e < 4; ++e) bias[e] = (bf16)0.f;
      if (a.bias && n_ok) bias = *reinterpret_cast<const bf16x4*>(a.bias + n);
    }
    if constexpr (HAS_LOADS) issue<0>();
    asm volatile("" ::: "memory");   // (not put off behind the slices)
  }
  template <int idx> __device__ __forceinline__ void finish(const float* stage, const float (&bias_v)[4], float (&cs)[4]) {
    constexpr int it0 = (idx % BPP) * UB;
    Batch& t = bt[idx & 1];
    f32x4 sv[UB];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int row_ = (it0 + u) * RPI + rd_row, row = EXACT ? row_ : min(row_, RP - 1);
      sv[u] = *reinterpret_cast<const f32x4*>(stage + Staged<WN>::slot(row, rd_chunk));
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      if (!t.ok[u]) continue;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = sv[u][e] + bias_v[e];
      if constexpr (EPI == EPI_ACCUM) {
        f32x4 c;
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = t.in32[u][e] + v[e];
        store_once<ONCE>(reinterpret_cast<f32x4*>(static_cast<float*>(a.C) + t.o[u]), c);
      } else if constexpr (GELU) {
        using T16 = std::conditional_t<OUT16, f16, bf16>;
        typedef T16 t16x4 __attribute__((ext_vector_type(4)));
        t16x4 uq, gq;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uq[e] = from_f32<T16>(v[e]);
          // g is the GeLU of u AS STORED, so that a backward pass that recomputes g from
          // the stashed u gets the same bits
          gq[e] = from_f32<T16>(gelu_f<EPI == EPI_GELU_TANH ? 0 : 1>((float)uq[e]));
        }
        store_once<ONCE>(reinterpret_cast<t16x4*>(static_cast<T16*>(a.C) + t.o[u]), uq);
        *reinterpret_cast<t16x4*>(reinterpret_cast<T16*>(a.gelu_out) + t.o[u]) = gq;
      } else {
        if constexpr (DGELU) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] *= gelu_grad_f<EPI == EPI_DGELU_TANH ? 0 : 1>((float)t.in16[u][e]);
        }
        if constexpr (EPI == EPI_BIAS_RES) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += (float)t.in16[u][e];
        }
        if constexpr (RES32) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += t.in32[u][e];
        }
        if constexpr (EPI == EPI_BIAS_RES32_OUT32) {
          f32x4 out;
#pragma unroll
          for (int e = 0; e < 4; ++e) out[e] = v[e];
          *reinterpret_cast<f32x4*>(static_cast<float*>(a.C) + t.o[u]) = out;
        } else if constexpr (OUT16 && EPI == EPI_BIAS) {
          f16x4 out;
#pragma unroll
          for (int e = 0; e < 4; ++e) out[e] = sat_f16(v[e]);
          *reinterpret_cast<f16x4*>(static_cast<f16*>(a.C) + t.o[u]) = out;
        } else {
          bf16x4 out;
#pragma unroll
          for (int e = 0; e < 4; ++e) out[e] = (bf16)v[e];
          *reinterpret_cast<bf16x4*>(static_cast<bf16*>(a.C) + t.o[u]) = out;
          if constexpr (DGELU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) cs[e] += v[e];
          }
        }
      }
    }
  }
  // stage: the wave's staged rows, pass by pass at the same place (write_pass(pass))
  // cs: GeLU' epilogue: on return, lanes < WN/4 hold the column sums of their four columns
  template <class StageWriter> __device__ __forceinline__ void run(StageWriter&& write_pass, const float* stage, float (&cs)[4], int lane) {
    float bias_v[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (BIAS) {
#pragma unroll
      for (int e = 0; e < 4; ++e) bias_v[e] = (float)bias[e];
    }
    static_for<NBATCH>([&](auto idx_c) {
      constexpr int idx = decltype(idx_c)::value;
      if constexpr (idx % BPP == 0) {
        write_pass(std::integral_constant<int, idx / BPP>{});
        // LDS operations of one wave complete in order: no wait is needed between the
        // writes above and the reads below, only that the compiler keeps their order
        asm volatile("" ::: "memory");
      }
      if constexpr (HAS_LOADS) {
        if constexpr (idx + 1 < NBATCH) issue<idx + 1>();
      } else {
        issue<idx>();
      }
      finish<idx>(stage, bias_v, cs);
    });
    if constexpr (DGELU) {
      // lanes CW apart hold the same columns of different rows
      if constexpr (FULL) {
#pragma unroll
        for (int off = CW; off < 64; off <<= 1)
#pragma unroll
          for (int e = 0; e < 4; ++e) cs[e] += __shfl_xor(cs[e], off);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float s = cs[e];
#pragma unroll
          for (int r = 1; r < RPI; ++r) s += __shfl(cs[e], (lane + r * CW) & 63);
          cs[e] = s;   // valid in lanes < CW
        }
      }
    }
  }
};

enum GemmForm { FORM_NT = 0, FORM_NN = 1, FORM_TN = 2 };

// F16: both operands hold fp16 values (A an activation stored in fp16, B the fp16 image of a
// weight); the f16 form of the matrix instruction is used and the 16-bit outputs are fp16.
// id: the workgroup's place among the product's tiles; lds: kernel's pipeline memory (gemm_lds_bytes()).
template <int MB, int NB, int BK, int NS> constexpr int gemm_lds_bytes() { return NS * 32 * (MB + NB) * BK * 2; }
template <typename P> __device__ __forceinline__ P* after(P* p, size_t bytes) {
  return (P*)((const char*)p + bytes);   // (by way of an integer it would no longer count as global memory)
}
template <int EPI, int FORM, bool F16, int MB, int NB, int BK, int NS>
__device__ __forceinline__ void gemm_tile(MfmaArgs a, int id, char* const lds) {
  constexpr bool A_KM = FORM == FORM_TN, B_KM = FORM != FORM_NT;
  constexpr int NW = 4, WM = 16 * MB, WN = 16 * NB, BM = 2 * WM, BN = 2 * WN, KS = BK / 32;
  using OpA = Operand<BM, BK, A_KM>;
  using OpB = Operand<BN, BK, B_KM>;
  constexpr int A_BYTES = OpA::BYTES, STAGE = A_BYTES + OpB::BYTES, RB = BK * 2, LDS_BYTES = NS * STAGE;
  constexpr int NIA = OpA::NI, N_DMA = NIA + OpB::NI;
  static_assert((KS == 1 || KS == 2) && LDS_BYTES <= 160 * 1024, "shape of the pipeline");
  static_assert(LDS_BYTES == gemm_lds_bytes<MB, NB, BK, NS>(), "pipeline memory");
  const uint32_t lds_base = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)lds;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / 2, wn = wave % 2;

  const int tiles_m1 = (a.M + BM - 1) / BM, tiles_m = tiles_m1 * (FORM == FORM_TN ? 1 : a.batch), tiles_n = (a.N + BN - 1) / BN;
  const int nb = tiles_m * tiles_n;
  {   // contiguous range of tiles per XCD (the first nb % 8 of them hold one more)
    const int x = id & 7, q = nb >> 3, r = nb & 7;
    id = x * q + min(x, r) + (id >> 3);
  }
  constexpr int GROUP = 4;
  const int per_group = GROUP * tiles_n;
  const int grp = id / per_group, first_m = grp * GROUP;
  const int gsz = min(tiles_m - first_m, GROUP);
  const int tm_i = first_m + (id % per_group) % gsz, tn_i = (id % per_group) / gsz;
  int tm = tm_i;   // tile row in its product
  if constexpr (FORM != FORM_TN) {
    if (a.batch > 1) {
      const int mb = __builtin_amdgcn_readfirstlane(tm_i / tiles_m1);
      tm = tm_i - mb * tiles_m1;
      a.A = after(a.A, mb * a.stride_a);
      a.C = after(static_cast<char*>(a.C), mb * a.stride_b);
      a.gelu_out = after(a.gelu_out, mb * a.stride_b);
      a.residual = after(static_cast<const char*>(a.residual), mb * (size_t)a.stride_r * 16);
      a.dgelu_u = after(a.dgelu_u, mb * (size_t)a.stride_r * 16);
    }
  }
  const int m0 = tm * BM, n0 = tn_i * BN;
  constexpr int PITCH = Staged<WN>::PITCH;
  constexpr int FIT = LDS_BYTES / NW / (PITCH * 4);        // rows of the wave's block that fit its LDS share
  constexpr int RP = FIT >= WM ? WM : (FIT >= 64 && WM % 64 == 0 ? 64 : 32);
  static_assert(FIT >= RP && WM % RP == 0, "epilogue staging does not fit");
  using Epi = GemmEpi<EPI, F16, WM, WN, RP>;
  Epi epi(a, m0 + wm * WM, n0 + wn * WN, lane);
  if constexpr (Epi::EARLY) epi.begin();
  const int sps = a.K / BK, nk = sps * (FORM == FORM_TN ? a.batch : 1);     // slices per K segment, in all

  const size_t lda = A_KM ? (size_t)a.M : (size_t)a.K, ldb = B_KM ? (size_t)a.N : (size_t)a.K;
  OpA opA;
  OpB opB;
  opA.init(m0, a.M, lda, wave, lane, false);
  opB.init(n0, a.N, ldb, wave, lane, a.b_img);

  // K-contiguous: fragment of 16 rows x 32 k: lane reads chunk 4*step + lane>>4 of row lane&15 (the
  // swizzle has period 16 rows)
  int kc_off[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    kc_off[ks] = (lane & 15) * RB + (((4 * ks + (lane >> 4)) ^ swz_kc(lane & 15)) << 4);
  const char* fragA = lds + (A_KM ? 0 : wm * WM * RB);
  const char* fragB = lds + A_BYTES + (B_KM ? 0 : wn * WN * RB);
  // K-major: transposing read t (0, 1) of block rb fetches k-rows 8*(lane>>4) + 4t + 0..3 of the
  // block's 16 columns; the lane supplies the address of k-row +(lane&15)>>2, 8-byte piece lane&3
  int rdA[A_KM ? 2 : 1][A_KM ? MB : 1], rdB[B_KM ? 2 : 1][B_KM ? NB : 1];
  if constexpr (B_KM) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int k = 8 * (lane >> 4) + 4 * t + ((lane & 15) >> 2);
      if constexpr (A_KM) {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) rdA[t][rb] = OpA::unit_off(k, wm * WM + rb * 16) + (lane & 3) * 8;
      }
#pragma unroll
      for (int rb = 0; rb < NB; ++rb) rdB[t][rb] = OpB::unit_off(k, wn * WN + rb * 16) + (lane & 3) * 8;
    }
  }
  auto frag_a = [&](int stage, int ks, int rb) -> bf16x8 {
    if constexpr (!A_KM) return *reinterpret_cast<const bf16x8*>(fragA + stage * STAGE + rb * 16 * RB + kc_off[ks]);
    else {
      const char* p = fragA + stage * STAGE + ks * 32 * OpA::ROWB;
      return tr_pair(p + rdA[0][rb], p + rdA[1][rb]);
    }
  };
  auto frag_b = [&](int stage, int ks, int rb) -> bf16x8 {
    if constexpr (!B_KM) return *reinterpret_cast<const bf16x8*>(fragB + stage * STAGE + rb * 16 * RB + kc_off[ks]);
    else {
      const char* p = fragB + stage * STAGE + ks * 32 * OpB::ROWB;
      return tr_pair(p + rdB[0][rb], p + rdB[1][rb]);
    }
  };
  bf16x8 fa[2][MB], fb[2][NB];

  static_for<MB * NB>([&](auto b_c) { agpr_zero4<4 * decltype(b_c)::value>(); });

  // The slice being fetched: its base addresses, advanced with wave-uniform arithmetic, and its place
  // in its segment (K-major operands); past the end the last slice is fetched again (redundant,
  // branch-free loop).
  const size_t step_a = A_KM ? (size_t)BK * lda : (size_t)BK;
  const size_t step_b = B_KM ? (size_t)BK * ldb : (a.b_img ? (size_t)256 * BK : (size_t)BK);
  int fill_left = nk - 1, fill_in_seg = 0;
  const bf16* fill_a = a.A;
  const bf16* fill_b = a.B;
  auto advance_fill = [&]() {
    if (fill_left > 0) {
      --fill_left;
      fill_a += step_a;
      fill_b += step_b;
      if constexpr (A_KM) {
        if (++fill_in_seg == sps) {
          fill_in_seg = 0;
          fill_a += a.stride_a - sps * step_a;
          fill_b += a.stride_b - sps * step_b;
        }
      }
    }
  };
  auto dma = [&](int stage, int i) {   // DMA instruction i of the slice: A first, then B
    if (i < NIA) opA.issue(fill_a, lds_base + stage * STAGE, wave, i);
    else opB.issue(fill_b, lds_base + stage * STAGE + A_BYTES, wave, i - NIA);
  };
  // Stage t % NS is free once every fragment of slice t is in registers, i.e. at the wait in front
  // of slice t's last step: from there on slice t + NS is copied into it -- in the last step (KS = 1),
  // or half in the last step and half in the first step of slice t + 1 (KS > 1, three or more stages).
  constexpr int D0 = KS == 1 || NS == 2 ? N_DMA : N_DMA / 2;     // DMA instructions of the last step
#pragma unroll
  for (int s0 = 0; s0 < NS; ++s0) {
#pragma unroll
    for (int i = 0; i < (s0 == NS - 1 ? D0 : N_DMA); ++i) dma(s0, i);
    if (D0 == N_DMA || s0 < NS - 1) advance_fill();
  }
  wait_dma_and_barrier<(NS - 2) * N_DMA + D0>();   // slice 0 has landed
#pragma unroll
  for (int u = 0; u < MB; ++u) fa[0][u] = frag_a(0, 0, u);
#pragma unroll
  for (int u = 0; u < NB; ++u) fb[0][u] = frag_b(0, 0, u);

  // One k = 32 step out of fragment buffer `cur`: matrix instructions with the fragments of the
  // next step (step ks_next of stage st_next) and DMA instructions [d_lo, d_hi) spread evenly between.
  auto step = [&](auto cur_c, auto st_next_c, auto ks_next_c, auto st_fill_c, auto lo_c, auto hi_c) {
    constexpr int cur = decltype(cur_c)::value, nxt = cur ^ 1, st_next = decltype(st_next_c)::value;
    constexpr int ks_next = decltype(ks_next_c)::value, st_fill = decltype(st_fill_c)::value;
    constexpr int d_lo = decltype(lo_c)::value, nd = decltype(hi_c)::value - d_lo, NBLK = MB * NB, NF = MB + NB;
    static_for<NBLK>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value, ib = i / NB, j0 = i % NB, jb = (ib & 1) ? NB - 1 - j0 : j0;
      // (block columns run forwards in even block rows and backwards in odd ones, so that exactly
      // one operand changes from one instruction to the next)
      mfma16_at<4 * (NB * ib + jb), F16>(fb[cur][jb], fa[cur][ib]);
      constexpr int f0 = i * NF / NBLK, f1 = (i + 1) * NF / NBLK, e0 = i * nd / NBLK, e1 = (i + 1) * nd / NBLK;
      if constexpr (f1 > f0 || e1 > e0) {
        __builtin_amdgcn_sched_barrier(0);
        static_for<f1 - f0>([&](auto f_c) {
          constexpr int f = f0 + decltype(f_c)::value;
          if constexpr (f < MB) fa[nxt][f] = frag_a(st_next, ks_next, f);
          else fb[nxt][f - MB] = frag_b(st_next, ks_next, f - MB);
        });
        static_for<e1 - e0>([&](auto e_c) { dma(st_fill, d_lo + e0 + decltype(e_c)::value); });
        __builtin_amdgcn_sched_barrier(0);
      }
    });
  };
  // unrolled over the ring, twice where the register buffers (which alternate per step) need it
  constexpr int UNROLL = KS == 1 && NS % 2 == 1 ? 2 * NS : NS;
  for (int kt = 0; kt < nk; kt += UNROLL) {
    static_for<UNROLL>([&](auto u_c) {
      constexpr int u = decltype(u_c)::value, r = u % NS, st_next = (r + 1) % NS, st_prev = (r + NS - 1) % NS;
      using std::integral_constant;
      constexpr integral_constant<int, r> r_c{};
      if (kt + u < nk) {
        if constexpr (KS == 2) {   // the first step finishes the copy begun in the slice before
          step(integral_constant<int, 0>{}, r_c, integral_constant<int, 1>{}, integral_constant<int, st_prev>{},
               integral_constant<int, D0>{}, integral_constant<int, N_DMA>{});
          if constexpr (D0 < N_DMA) advance_fill();
        }
        // slice t+1 has landed; every fragment of slice t is in registers (of every wave)
        wait_dma_and_barrier<(NS - 2) * N_DMA>();
        step(integral_constant<int, KS == 1 ? (u & 1) : 1>{}, integral_constant<int, st_next>{}, integral_constant<int, 0>{}, r_c,
             integral_constant<int, 0>{}, integral_constant<int, D0>{});
        if constexpr (D0 == N_DMA) advance_fill();
      }
    });
  }
  // no DMA may still be writing LDS when the staging starts; the matrix pipeline must have
  // drained before the accumulators are read (the compiler does not know they were written)
  asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
  __syncthreads();

  // rows [pass*RP, +RP) of the wave's block -> its staging area
  auto stage_rows = [&](auto pass_c, auto rp_c, float* stg) {
    constexpr int pass = decltype(pass_c)::value, BI = decltype(rp_c)::value / 16;   // block rows per pass
    static_for<BI * NB>([&](auto b_c) {
      constexpr int ii = decltype(b_c)::value / NB, jb = decltype(b_c)::value % NB;
      constexpr int R = 4 * (NB * (pass * BI + ii) + jb);
      f32x4 v;
      v[0] = agpr_read<R>();
      v[1] = agpr_read<R + 1>();
      v[2] = agpr_read<R + 2>();
      v[3] = agpr_read<R + 3>();
      *reinterpret_cast<f32x4*>(stg + Staged<WN>::slot(ii * 16 + (lane & 15), jb * 4 + (lane >> 4))) = v;
    });
  };
  // GeLU' epilogue: the lane's share of the column sums of C, before rounding to bf16 (the bias
  // gradient of the linear layer whose output gradient this product forms)
  float cs[4] = {0.f, 0.f, 0.f, 0.f};
  float* const stg = reinterpret_cast<float*>(lds) + wave * (RP * PITCH);
  if constexpr (!Epi::EARLY) epi.begin();
  epi.run([&](auto pass_c) { stage_rows(pass_c, std::integral_constant<int, RP>{}, stg); }, stg, cs, lane);
  if constexpr ((EPI & ~EPI_ONCE) == EPI_DGELU_TANH || (EPI & ~EPI_ONCE) == EPI_DGELU_ERF) {
    const int n = n0 + wn * WN + lane * 4;
    if (a.colsum && lane < WN / 4 && n < a.N) {
      f32x4 out;
#pragma unroll
      for (int e = 0; e < 4; ++e) out[e] = cs[e];
      *reinterpret_cast<f32x4*>(a.colsum + (size_t)(tm_i * 2 + wm) * a.N + n) = out;
    }
  }
}

// Waves per SIMD the registers have to allow: two where half of the LDS holds a ring of the largest tile that two
// workgroups in a unit can have (256x128: 128 accumulators and at most 128 other registers); the smaller ones
// need no limit.
template <int MB, int NB, int BK, int NS> constexpr int gemm_waves() {
  return MB * NB >= 32 && gemm_lds_bytes<MB, NB, BK, NS>() <= 80 * 1024 ? 2 : 1;
}
template <int EPI, int FORM, bool F16, int MB, int NB, int BK, int NS>
__global__ __launch_bounds__(256, (gemm_waves<MB, NB, BK, NS>())) void gemm_mi16_kernel(const MfmaArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds[gemm_lds_bytes<MB, NB, BK, NS>()];
  gemm_tile<EPI, FORM, F16, MB, NB, BK, NS>(a, blockIdx.x, lds);
}

// Several weight gradients in one launch, one after the other in the order of the workgroups: their
// last, partly filled rounds of tiles run into the next product's first.
// The workgroups from `blocks` on add up partial column sums: alone these are a launch of some microseconds whatever
// their size, here they fill units that the last round of tiles leaves idle.  In a launch of their own | here, us a step:
// 128 fp32 tokens 128 wide 67.3 | 64.8, 192 tokens 320 wide 299.7 | 290.3, 4096 tokens 1024 wide 1987 | 1970, 2048 tokens
// 5120 wide (2080 workgroups of sums) no difference.
struct WgradGroup {
  MfmaArgs p[kMaxWgrads];
  int first[kMaxWgrads];   // first workgroup of a product
  int blocks;              // of the products
  ReduceArgs<kMaxReduceSegs> sums;
};
template <int EPI, int FORM, bool F16, int MB, int NB, int BK, int NS>
__global__ __launch_bounds__(256, (gemm_waves<MB, NB, BK, NS>())) void gemm_mi16_group_kernel(const WgradGroup g) {
  __shared__ __attribute__((aligned(1024))) char lds[gemm_lds_bytes<MB, NB, BK, NS>()];
  if ((int)blockIdx.x >= g.blocks) {
    static_assert(sizeof(float[1][32][33]) <= sizeof(lds), "room for the sums");
    reduce_columns<kMaxReduceSegs, 1>(g.sums, blockIdx.x - g.blocks, reinterpret_cast<float(*)[32][33]>(lds));
    return;
  }
  int k = 0;
#pragma unroll
  for (int i = 1; i < kMaxWgrads; ++i)
    if ((int)blockIdx.x >= g.first[i]) k = i;
  gemm_tile<EPI, FORM, F16, MB, NB, BK, NS>(g.p[k], blockIdx.x - g.first[k], lds);
}

// The kinds and tiles that have a form for MfmaArgs::once.  Tiles below 128x128 have none: they are for smaller matrices, but for
// the GeLU' product of a pass over a window, which keeps the tile of one micro-batch.
template <int EPI, int MB, int NB> constexpr bool has_once() {
  return MB * NB >= 16 && (EPI == EPI_ACCUM || EPI == EPI_GELU_TANH || EPI == EPI_GELU_ERF || EPI == EPI_DGELU_TANH || EPI == EPI_DGELU_ERF);
}
template <int EPI, int FORM, bool F16, int MB, int NB, int BK, int NS>
hipError_t launch_mi16(const MfmaArgs& a, hipStream_t st) {
  if constexpr (has_once<EPI, MB, NB>()) {
    if (a.once) return launch_mi16<EPI | EPI_ONCE, FORM, F16, MB, NB, BK, NS>(a, st);
  }
  if (a.b_img && BK != kImageK) return hipErrorInvalidValue;
  const int tiles = (FORM == FORM_TN ? 1 : a.batch) * ((a.M + 32 * MB - 1) / (32 * MB)) * ((a.N + 32 * NB - 1) / (32 * NB));
  hipLaunchKernelGGL((gemm_mi16_kernel<EPI, FORM, F16, MB, NB, BK, NS>), dim3(tiles), dim3(256), 0, st, a);
  return hipGetLastError();
}

// One product alone takes the plain kernel: a quarter of the arguments, 0.4 us less to launch.
template <int MB, int NB, int BK, int NS>
hipError_t launch_group(const MfmaArgs* a, int n, const ReduceSeg* sums, int n_sums, hipStream_t st) {
  if (n == 1 && n_sums == 0) return launch_mi16<EPI_ACCUM, FORM_TN, false, MB, NB, BK, NS>(a[0], st);
  WgradGroup g{};
  int blocks = 0;
  for (int i = 0; i < kMaxWgrads; ++i) {
    g.p[i] = a[i < n ? i : 0];
    g.first[i] = i < n ? blocks : 0x7fffffff;      // (never reached)
    if (i < n) blocks += ((a[i].M + 32 * MB - 1) / (32 * MB)) * ((a[i].N + 32 * NB - 1) / (32 * NB));
  }
  g.blocks = blocks;
  blocks += reduce_layout<kMaxReduceSegs>(sums, n_sums, &g.sums);
  if constexpr (has_once<EPI_ACCUM, MB, NB>()) {
    if (a[0].once) {
      hipLaunchKernelGGL((gemm_mi16_group_kernel<EPI_ACCUM | EPI_ONCE, FORM_TN, false, MB, NB, BK, NS>), dim3(blocks), dim3(256), 0, st, g);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((gemm_mi16_group_kernel<EPI_ACCUM, FORM_TN, false, MB, NB, BK, NS>), dim3(blocks), dim3(256), 0, st, g);
  return hipGetLastError();
}

template <int EPI, int FORM, bool F16, int MB, int NB> hipError_t launch_ring(const MfmaArgs& a, hipStream_t st) {
  const long tiles = (long)a.batch * ((a.M + 32 * MB - 1) / (32 * MB)) * ((a.N + 32 * NB - 1) / (32 * NB));
  return two_stages(tiles, a.K) ? launch_mi16<EPI, FORM, F16, MB, NB, 64, 2>(a, st) : launch_mi16<EPI, FORM, F16, MB, NB, 64, 4>(a, st);
}
// Six stages instead of four gain nothing at 128x64 and 64x32 (two layers of 192 rows, 320 wide: 335
// against 338 us a step; 512 rows, 1024 wide, four chunks: 4999 against 5008 us).
template <int EPI, int FORM, bool F16 = false> hipError_t launch_tile(Tile tile, const MfmaArgs& a, hipStream_t st) {
  switch (tile) {
    case TILE_256x256: return launch_mi16<EPI, FORM, F16, 8, 8, 64, 2>(a, st);
    case TILE_256x192: return launch_mi16<EPI, FORM, F16, 8, 6, 64, 2>(a, st);
    case TILE_256x160: return launch_mi16<EPI, FORM, F16, 8, 5, 64, 3>(a, st);
    case TILE_192x192: return launch_mi16<EPI, FORM, F16, 6, 6, 64, 3>(a, st);
    case TILE_256x128: return launch_mi16<EPI, FORM, F16, 8, 4, 64, 3>(a, st);
    case TILE_128x128: return launch_ring<EPI, FORM, F16, 4, 4>(a, st);
    case TILE_128x64: return launch_ring<EPI, FORM, F16, 4, 2>(a, st);
    case TILE_64x64: return launch_mi16<EPI, FORM, F16, 2, 2, 64, 4>(a, st);
    case TILE_64x32: return launch_mi16<EPI, FORM, F16, 2, 1, 64, 4>(a, st);
    default: return hipErrorInvalidValue;
  }
}
// Weight gradients, two K-major operands: the two widest tiles take slices of 32 in four or five stages.
// Their rows are whole lines at any depth, and the transposing reads leave no room for a copy as
// bursty as two stages of 64 (4096^3: 115 against 118 us; 3968x6144x2048 with 192 columns: 109 against
// 117 us).  With a K-contiguous operand two stages of 64 win (97 against 102 us; 84 against 94 us).
// 256x128 and 128x128 take slices of 32 in half of the LDS: two workgroups share a unit, and one's read-modify-write
// of the fp32 matrix, a fifth of a lone workgroup's time, runs under the other's slices.  In slices of 64 and all
// of the LDS | this, us: 256x128 6144x4096, K = 2048 113 | 98, 4096x2048 (one round of 256) 37.1 | 36.6, 3072x3072,
// K = 4096 106 | 89; 128x128 4096x4096, K = 1024 57 | 45, 3072x2048, K = 4096 62 | 56, 4096x1024 (one round)
// 37.1 | 36.5; 128x128 with two slices of 64: 4 % slower than with four of 64, five of 32: within 2 % of four.
inline hipError_t launch_wgrads(Tile tile, const MfmaArgs* a, int n, const ReduceSeg* sums, int n_sums, hipStream_t st) {
  switch (tile) {
    case TILE_256x256: return launch_group<8, 8, 32, 4>(a, n, sums, n_sums, st);
    case TILE_256x192: return launch_group<8, 6, 32, 5>(a, n, sums, n_sums, st);
    case TILE_256x160: return launch_group<8, 5, 64, 3>(a, n, sums, n_sums, st);
    case TILE_192x192: return launch_group<6, 6, 64, 3>(a, n, sums, n_sums, st);
    case TILE_256x128: return launch_group<8, 4, 32, 3>(a, n, sums, n_sums, st);
    case TILE_128x128: return launch_group<4, 4, 32, 4>(a, n, sums, n_sums, st);
    case TILE_128x64: return launch_group<4, 2, 64, 4>(a, n, sums, n_sums, st);
    case TILE_64x64: return launch_group<2, 2, 64, 4>(a, n, sums, n_sums, st);
    case TILE_64x32: return launch_group<2, 1, 64, 4>(a, n, sums, n_sums, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace
}  // namespace gpts

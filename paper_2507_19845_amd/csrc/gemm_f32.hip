// fp32 matrix products on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 multiply-add, fp32
// accumulation), for fp32 stages whose operands are 16-byte aligned with widths that are
// multiples of 4; gemm_simple.hip takes the rest.  The three forms of the stage:
//   NT  C = A[M,K] B[N,K]^T    NN  C = A[M,K] B[K,N]    TN  C += A[K,M]^T B[K,N]
//
// A wave owns a 32 x 32 block of C, 2 x 2 blocks of 16 x 16 whose rows and columns are
// INTERLEAVED: block b holds the rows (columns) 2*idx + b.  A lane then gets its two blocks'
// elements of a K-major operand ([k][rows], as it sits in memory) with one 8-byte LDS read, and
// the eight accumulator values it holds of one row of C are eight consecutive columns.  A
// K-contiguous operand gives a lane four consecutive k with one 16-byte read, i.e. four matrix
// steps: in step s lane group g = lane/16 multiplies k = 4g + s, for both kinds of operand.
//
// Three arrangements of the waves:
//   2 x 2 x 1  a 64 x 64 tile of C, slices of 32 k
//   1 x 1 x 8  a 32 x 32 tile, slices of 128 k of which each wave multiplies an eighth; the eight
//              partial tiles are added through LDS in fixed order.  Four times the tiles, two of them and so
//              four waves per SIMD in a unit: the form for products that do not fill the chip.
//   1 x 1 x 4  the same with four waves and slices of 64 k, for weight gradients: the padded tiles of two
//              K-major operands leave room for one workgroup of eight waves in a unit, for four of these.
// Slices travel global -> registers -> LDS, four slices ahead in registers (two of the eight waves' slices, which
// are twice as long) and double buffered in LDS, one barrier per slice.
// Bound: the fp32 matrix pipe (157 TFLOP/s) where there are tiles enough, below that launch, first slice and
// the sum of the partial tiles, about 5 us.  us, two slices ahead and four waves to a narrow tile | now: NT
// 4096x4096x4096 1131 (121 TFLOP/s) | 997 (138); NN 999x512x2048 30.6 | 26.5, 999x512x1536 23.3 | 20.7; NT
// 300x384x1536 13.2 | 10.5, 999x512x512 9.2 | 9.6, 128x128x128 8.0 | 7.6; the four weight gradients of 512 and 2048
// columns over 999 tokens 77 | 71.  Four of the eight waves' slices ahead: 27.4 and 21.9, 10.2; weight gradients in
// 64 x 64 tiles of four waves that split the contraction: 71.  Against gemm_simple_kernel (64 x 64 x 16, fp32 FMA):
// NN 999x512x2048 243 us, NT 128x128x128 11.6.
#include "reduce.hpp"

namespace gpts {
namespace {

enum { F32_PLAIN = 0, F32_GELU_TANH, F32_GELU_ERF, F32_DGELU_TANH, F32_DGELU_ERF, F32_ACCUM };

struct F32Args {
  const float* A;
  const float* B;
  float* C;
  int M, N, K;
  const float* bias;
  const float* residual;
  float* gelu_out;
  const float* dgelu_u;
};

// One operand's tile of R rows x BK k, NT threads: global loads into registers, LDS stores, fragment reads.
template <int R, int BK, bool KMAJOR, int NT> struct F32Operand {
  static constexpr int PER = R * BK / 4 / NT;               // 16-byte pieces per thread
  static constexpr int CPR = KMAJOR ? R / 4 : BK / 4;       // pieces per row of the LDS tile
  // K-major rows are padded by 8 floats so that the four k-rows a wave reads together lie 32
  // banks apart; K-contiguous rows are swizzled instead (place())
  static constexpr int PITCH = KMAJOR ? R + 8 : BK;
  static constexpr int FLOATS = (KMAJOR ? BK : R) * PITCH;
  static_assert(R * BK / 4 % NT == 0, "whole pieces per thread");
  // longest row (elements) for which the 32-bit byte offsets below hold: a slice is BK rows (K-major) or R of them
  static constexpr int MAX_ROW = (1 << 30) / (KMAJOR ? BK : R);

  const float* base;       // the tile's first row, slice 0 (wave-uniform)
  uint32_t off[PER];       // bytes from there to this thread's pieces
  uint32_t off_last[PER];  // the same in a last slice that the contraction ends in: pieces past the end read the last
  int k_of[PER];           // their first k
  int dst[PER];            // LDS offsets (floats)

  // LDS offset (floats) of a piece of a K-contiguous row.  A wave reads the rows 2i + b (i = 0..15), at one piece
  // per 16 lanes; a 16-byte read serves lanes {0-3, 12-15, 20-27} of a half wave together, then the others: those
  // of eight i at one piece and of the other eight at the next.  Rows of 16 or 32 pieces fill the 64 banks: XOR with i.
  // Rows of eight fill half of them: the even rows lie before the odd ones, so that i & 1 is the half, XOR with i / 2.
  static __device__ __forceinline__ int place(int row, int piece) {
    if constexpr (CPR >= 16) return row * PITCH + (piece ^ ((row >> 1) & 15)) * 4;
    else return ((row & 1) * (R / 2) + (row >> 1)) * PITCH + (piece ^ ((row >> 2) & 7)) * 4;
  }
  __device__ __forceinline__ void init(const float* X, int r0, int rtotal, int K) {
    base = KMAJOR ? X + r0 : X + (size_t)r0 * K;
    const int rest = K - (K - 1) / BK * BK;                         // k of the last slice
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int idx = threadIdx.x + NT * p, row = idx / CPR, c = idx % CPR;
      if constexpr (KMAJOR) {
        const int col = min(c * 4, rtotal - r0 - 4);               // past the edge: any valid column
        off[p] = ((uint32_t)row * rtotal + col) * 4;
        off_last[p] = ((uint32_t)min(row, rest - 1) * rtotal + col) * 4;
        k_of[p] = row;
        dst[p] = row * PITCH + c * 4;
      } else {
        const int lr = min(row, rtotal - 1 - r0);
        off[p] = ((uint32_t)lr * K + c * 4) * 4;
        off_last[p] = ((uint32_t)lr * K + min(c * 4, rest - 4)) * 4;
        k_of[p] = c * 4;
        dst[p] = place(row, c);
      }
    }
  }
  // pieces of slice kt (last: the last one)
  __device__ __forceinline__ void load(f32x4 (&v)[PER], int kt, bool last, int rtotal) const {
    const char* const b = reinterpret_cast<const char*>(base + (KMAJOR ? (size_t)kt * BK * rtotal : (size_t)kt * BK));
#pragma unroll
    for (int p = 0; p < PER; ++p) v[p] = *reinterpret_cast<const f32x4*>(b + (last ? off_last[p] : off[p]));
  }
  // k past the end of the contraction becomes zero (in both operands, so nothing is multiplied by what
  // lies there); left: k from this slice's first to the end
  __device__ __forceinline__ void cut(f32x4 (&v)[PER], int left) const {
#pragma unroll
    for (int p = 0; p < PER; ++p)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[p][e] = k_of[p] < left ? v[p][e] : 0.f;
  }
  __device__ __forceinline__ void store(const f32x4 (&v)[PER], float* tile) const {
#pragma unroll
    for (int p = 0; p < PER; ++p) *reinterpret_cast<f32x4*>(tile + dst[p]) = v[p];
  }
  // the two blocks' fragments of the 16 k starting at k0 (a multiple of 16) for rows w0..w0+31:
  // f[b][s] = element (row w0 + 2*(lane%16) + b, k = k0 + 4*(lane/16) + s)
  __device__ __forceinline__ static void frag(float (&f)[2][4], const float* tile, int w0, int k0, int lane) {
    const int i = lane & 15, g = lane >> 4;
    if constexpr (KMAJOR) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const f32x2 v = *reinterpret_cast<const f32x2*>(tile + (k0 + 4 * g + s) * PITCH + w0 + 2 * i);
        f[0][s] = v[0];
        f[1][s] = v[1];
      }
    } else {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int row = w0 + 2 * i + b;
        const f32x4 v = *reinterpret_cast<const f32x4*>(tile + place(row, (k0 >> 2) + g));
#pragma unroll
        for (int s = 0; s < 4; ++s) f[b][s] = v[s];
      }
    }
  }
};

// Four columns of a row of C: what their epilogue reads is asked for in front of the slices (begin()), so that no memory
// latency follows the last one: a step of 128 tokens 128 wide 64.8 -> 63.6 us, of 999 tokens 512 wide 607 -> 605.
template <int EPI> struct F32Out {
  static constexpr bool GELU = EPI == F32_GELU_TANH || EPI == F32_GELU_ERF, DGELU = EPI == F32_DGELU_TANH || EPI == F32_DGELU_ERF;
  size_t o;
  bool ok;
  f32x4 bias, in, res;   // in: C of an accumulating product, u for GeLU'
  static __device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
  __device__ __forceinline__ void begin(const F32Args& a, int m, int n) {
    ok = m < a.M && n < a.N;
    o = (size_t)m * a.N + n;
    bias = in = res = f32x4{0.f, 0.f, 0.f, 0.f};
    if (!ok) return;
    if constexpr (EPI == F32_ACCUM) in = ld4(a.C + o);
    else if (a.bias) bias = ld4(a.bias + n);
    if constexpr (DGELU) in = ld4(a.dgelu_u + o);
    if constexpr (EPI != F32_ACCUM && !GELU) {
      if (a.residual) res = ld4(a.residual + o);
    }
  }
  __device__ __forceinline__ void store(const F32Args& a, f32x4 v) const {
    if (!ok) return;
    if constexpr (EPI == F32_ACCUM) {
      *reinterpret_cast<f32x4*>(a.C + o) = in + v;
    } else {
      if (a.bias) v += bias;
      if constexpr (GELU) {
        f32x4 gq;
#pragma unroll
        for (int e = 0; e < 4; ++e) gq[e] = gelu_f<EPI == F32_GELU_TANH ? 0 : 1>(v[e]);
        *reinterpret_cast<f32x4*>(a.C + o) = v;
        *reinterpret_cast<f32x4*>(a.gelu_out + o) = gq;
      } else {
        if constexpr (DGELU) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] *= gelu_grad_f<EPI == F32_DGELU_TANH ? 0 : 1>(in[e]);
        }
        if (a.residual) v += res;
        *reinterpret_cast<f32x4*>(a.C + o) = v;
      }
    }
  }
};

// The arrangement of a workgroup's WM x WN x WK waves; WK of them share the contraction.
template <int WM, int WN, int WK, bool A_KM, bool B_KM> struct F32Shape {
  static_assert(WK == 1 ? WM * WN == 4 : WM * WN == 1, "a split contraction has one tile");
  static constexpr int NT = 64 * WM * WN * WK, BM = 32 * WM, BN = 32 * WN, BK = WK == 1 ? 32 : 16 * WK;
  using OpA = F32Operand<BM, BK, A_KM, NT>;
  using OpB = F32Operand<BN, BK, B_KM, NT>;
  static constexpr int STAGE = OpA::FLOATS + OpB::FLOATS, LDS_FLOATS = 2 * STAGE;
  static_assert(WK == 1 || LDS_FLOATS >= WK * BM * BN, "the partial tiles fit");
};
constexpr int kMaxRow = 1 << 24;   // rows of A and B are shorter (gemm_f32_supported())
template <int WM, int WN, int WK, bool A_KM, bool B_KM, int EPI>
__device__ __forceinline__ void f32_tile(const F32Args& a, int tile_m, int tile_n, float* const lds) {
  using Shape = F32Shape<WM, WN, WK, A_KM, B_KM>;
  using OpA = typename Shape::OpA;
  using OpB = typename Shape::OpB;
  constexpr int BM = Shape::BM, BN = Shape::BN, BK = Shape::BK, KW = BK / WK, STAGE = Shape::STAGE;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  OpA opA;
  OpB opB;
  opA.init(a.A, m0, a.M, a.K);
  opB.init(a.B, n0, a.N, a.K);
  const int nk = (a.K + BK - 1) / BK;

  // acc[ib][jb][r] = C[2i + ib][2(4g + r) + jb] of the wave's block: columns 8g .. 8g+7 of a row
  const int i = lane & 15, g = lane >> 4;
  F32Out<EPI> out[WK == 1 ? 4 : 1];
  if constexpr (WK == 1) {
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q].begin(a, m0 + wm * 32 + 2 * i + (q >> 1), n0 + wn * 32 + 8 * g + 4 * (q & 1));
  } else if (WK == 4 || wave < 4) {   // the first four waves each store a quarter of the tile
    out[0].begin(a, m0 + 2 * i + (wave >> 1), n0 + 8 * g + 4 * (wave & 1));
  }
  asm volatile("" ::: "memory");   // (the loads are not put off behind the slices)

  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int AHEAD = WK == 8 ? 2 : 4;                      // slices in registers (an even number)
  f32x4 ra[AHEAD][OpA::PER], rb[AHEAD][OpB::PER];
  auto load = [&](int t, int r) {
    if (t < nk) {
      opA.load(ra[r], t, t == nk - 1, a.M);
      opB.load(rb[r], t, t == nk - 1, a.N);
    }
  };
  auto store = [&](int t, int r, float* stage) {
    if (t == nk - 1) {
      opA.cut(ra[r], a.K - t * BK);
      opB.cut(rb[r], a.K - t * BK);
    }
    opA.store(ra[r], stage);
    opB.store(rb[r], stage + OpA::FLOATS);
  };
  auto multiply = [&](const float* st) {
#pragma unroll
    for (int q = 0; q < KW / 16; ++q) {
      float fa[2][4], fb[2][4];
      OpA::frag(fa, st, wm * 32, wk * KW + q * 16, lane);
      OpB::frag(fb, st + OpA::FLOATS, wn * 32, wk * KW + q * 16, lane);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)   // operands swapped: a lane gets four columns of one row
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][s], fa[i][s], acc[i][j], 0, 0, 0);
    }
  };
#pragma unroll
  for (int t = 0; t < AHEAD; ++t) load(t, t);
  store(0, 0, lds);
  load(AHEAD, 0);
  __syncthreads();
  for (int t = 0; t < nk; t += AHEAD) {
#pragma unroll
    for (int h = 0; h < AHEAD; ++h) {
      // slice t+h lies in stage h % 2; slice t+h+1 goes from registers to the other stage (every wave
      // left that one before the last barrier)
      if (t + h < nk) {
        multiply(lds + (h & 1) * STAGE);
        if (t + h + 1 < nk) {
          store(t + h + 1, (h + 1) % AHEAD, lds + ((h + 1) & 1) * STAGE);
          load(t + h + 1 + AHEAD, (h + 1) % AHEAD);
        }
        __syncthreads();
      }
    }
  }

  auto half = [&](int ib, int h) {
    return f32x4{acc[ib][0][2 * h], acc[ib][1][2 * h], acc[ib][0][2 * h + 1], acc[ib][1][2 * h + 1]};
  };
  if constexpr (WK == 1) {
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int h = 0; h < 2; ++h) out[2 * ib + h].store(a, half(ib, h));
  } else {
    // the first four waves each add up and store one quarter of the tile (the loop's last barrier has freed the LDS)
    f32x4* part = reinterpret_cast<f32x4*>(lds);
#pragma unroll
    for (int q = 0; q < 4; ++q) part[(wave * 4 + q) * 64 + lane] = half(q >> 1, q & 1);
    __syncthreads();
    if (WK > 4 && wave >= 4) return;
    f32x4 v = part[wave * 64 + lane];
#pragma unroll
    for (int w = 1; w < WK; ++w) v += part[(w * 4 + wave) * 64 + lane];
    out[0].store(a, v);
  }
}

template <int WM, int WN, int WK, bool A_KM, bool B_KM, int EPI>
__global__ __launch_bounds__(64 * WM * WN * WK) void gemm_f32_kernel(const F32Args a) {
  __shared__ __attribute__((aligned(16))) float lds[F32Shape<WM, WN, WK, A_KM, B_KM>::LDS_FLOATS];
  f32_tile<WM, WN, WK, A_KM, B_KM, EPI>(a, blockIdx.y, blockIdx.x, lds);
}
// Several weight gradients in one launch.
struct F32Group {
  F32Args p[kMaxWgrads];
  int first[kMaxWgrads];   // first workgroup of a product
  int blocks;              // of the products; those from here on add up partial column sums
  ReduceArgs<kMaxReduceSegs> sums;
};
template <int WM, int WN, int WK> __global__ __launch_bounds__(256) void gemm_f32_group_kernel(const F32Group g) {
  using Shape = F32Shape<WM, WN, WK, true, true>;
  __shared__ __attribute__((aligned(16))) float lds[Shape::LDS_FLOATS];
  if ((int)blockIdx.x >= g.blocks) {
    static_assert(Shape::LDS_FLOATS >= 32 * 33, "room for the sums");
    reduce_columns<kMaxReduceSegs, 1>(g.sums, blockIdx.x - g.blocks, reinterpret_cast<float(*)[32][33]>(lds));
    return;
  }
  int k = 0;
#pragma unroll
  for (int i = 1; i < kMaxWgrads; ++i)
    if ((int)blockIdx.x >= g.first[i]) k = i;
  const int id = blockIdx.x - g.first[k], tiles_n = (g.p[k].N + Shape::BN - 1) / Shape::BN;
  f32_tile<WM, WN, WK, true, true, F32_ACCUM>(g.p[k], id / tiles_n, id % tiles_n, lds);
}

// 64 x 64 tiles, or 32 x 32 tiles with a split contraction?  The first take a step of time with every 256 of them, of
// which each compute unit has one more to do; the others a unit shares evenly, but for each multiply-add they move twice
// the bytes.  The estimates are fitted to products of 128 ... 768 tiles of 64 x 64 and K = 256 ... 2048, within 8 %.
// us, 64 / 32, NT (NN is within 5 %):     K = 256        512          2048
//   999x512, 128 tiles                    8.3 /  7.4   13.6 /  9.4   44.0 / 25.5
//   999x1024, 256                         8.4 / 10.0   13.5 / 15.1   44.4 / 43.8
//   999x1280, 320                        12.4 / 12.3   21.4 / 18.0   73.3 / 54.1
//   999x2048, 512                        12.8 / 18.1   21.7 / 26.8   73.9 / 84.1
//   1536x1536, 576                       17.3 / 20.1   29.4 / 29.8  101.7 / 94.6
// TN 1280x999, 320                       14.0 / 11.7   23.4 / 18.1   78.5 / 55.8;  1999x512, 512  14.7 / 16.3  24.0 / 25.8  79.0 / 82.4
bool use_wide(int form, int M, int N, int K) {
  const float n = (float)((M + 63) / 64) * (float)((N + 63) / 64), rounds = ceilf(n / 256.f), k = (float)K;
  const float narrow = 3.f + 0.0105f * n + (0.0016f + 6.95e-5f * n) * k;
  const float wide = form == 2 ? 2.9f + 1.2f * rounds + (0.009f + 0.0135f * rounds) * k
                               : 2.5f + 1.0f * rounds + (0.0065f + 0.0137f * rounds) * k;
  return wide < 0.97f * narrow;
}

template <bool A_KM, bool B_KM, int EPI> hipError_t launch_f32(const F32Args& a, hipStream_t st) {
  using Wide = F32Shape<2, 2, 1, A_KM, B_KM>;
  using Narrow = F32Shape<1, 1, 8, A_KM, B_KM>;
  static_assert(!A_KM && Wide::OpA::MAX_ROW >= kMaxRow && Wide::OpB::MAX_ROW >= kMaxRow && Narrow::OpA::MAX_ROW >= kMaxRow, "offsets fit");
  // (the narrow tile's slices of a K-major B are 128 rows: 2^23 columns)
  if ((B_KM ? a.N : a.K) > Narrow::OpB::MAX_ROW || use_wide(B_KM ? 1 : 0, a.M, a.N, a.K)) {
    hipLaunchKernelGGL((gemm_f32_kernel<2, 2, 1, A_KM, B_KM, EPI>), dim3((a.N + 63) / 64, (a.M + 63) / 64), dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL((gemm_f32_kernel<1, 1, 8, A_KM, B_KM, EPI>), dim3((a.N + 31) / 32, (a.M + 31) / 32), dim3(512), 0, st, a);
  }
  return hipGetLastError();
}

template <int WM, int WN, int WK>
hipError_t launch_f32_group(const F32Args* a, int n, const ReduceSeg* sums, int n_sums, hipStream_t st) {
  using Shape = F32Shape<WM, WN, WK, true, true>;
  static_assert(Shape::OpA::MAX_ROW >= kMaxRow && Shape::OpB::MAX_ROW >= kMaxRow, "offsets fit");
  F32Group g{};
  int blocks = 0;
  for (int i = 0; i < kMaxWgrads; ++i) {
    g.p[i] = a[i < n ? i : 0];
    g.first[i] = i < n ? blocks : 0x7fffffff;      // (never reached)
    if (i < n) blocks += ((a[i].M + Shape::BM - 1) / Shape::BM) * ((a[i].N + Shape::BN - 1) / Shape::BN);
  }
  g.blocks = blocks;
  blocks += reduce_layout<kMaxReduceSegs>(sums, n_sums, &g.sums);
  hipLaunchKernelGGL((gemm_f32_group_kernel<WM, WN, WK>), dim3(blocks), dim3(256), 0, st, g);
  return hipGetLastError();
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

// 16-byte pieces: every contiguous dimension a multiple of 4, every pointer 16-byte aligned; the
// grid's y dimension holds at most 65535 tile rows; offsets within a slice of a tile are 32 bits.
bool gemm_f32_supported(int form, int M, int N, int K, const void* A, const void* B, const void* C,
                        const GemmEpilogue& ep) {
  if (N >= kMaxRow || (form == 2 ? M : K) >= kMaxRow) return false;
  return N % 4 == 0 && (form == 2 ? M % 4 == 0 : K % 4 == 0) && M <= 32 * 65535 && aligned16(A) && aligned16(B) &&
         aligned16(C) && aligned16(ep.bias) && aligned16(ep.residual) && aligned16(ep.gelu_out) && aligned16(ep.dgelu_u);
}

hipError_t gemm_f32(int form, int M, int N, int K, const void* A, const void* B, void* C,
                    const GemmEpilogue& ep, hipStream_t st) {
  if (!gemm_f32_supported(form, M, N, K, A, B, C, ep)) return hipErrorInvalidValue;
  const F32Args a{(const float*)A, (const float*)B, (float*)C, M, N, K, (const float*)ep.bias, (const float*)ep.residual,
                  (float*)ep.gelu_out, (const float*)ep.dgelu_u};
  if (form == 0) {
    if (a.gelu_out) return ep.gelu_kind == 0 ? launch_f32<false, false, F32_GELU_TANH>(a, st) : launch_f32<false, false, F32_GELU_ERF>(a, st);
    return launch_f32<false, false, F32_PLAIN>(a, st);
  }
  if (form == 1) {
    if (a.dgelu_u) return ep.gelu_kind == 0 ? launch_f32<false, true, F32_DGELU_TANH>(a, st) : launch_f32<false, true, F32_DGELU_ERF>(a, st);
    return launch_f32<false, true, F32_PLAIN>(a, st);
  }
  const WgradItem w{M, N, A, B, (float*)C};
  return gemm_f32_wgrad_group(&w, 1, K, st);
}

// Each product keeps the tile it has alone (use_wide), so that its bits do not depend on its company.
hipError_t gemm_f32_wgrad_group(const WgradItem* items, int n, int K, hipStream_t st, const ReduceSeg* sums, int n_sums) {
  if (n < 1 || n > kMaxWgrads || !few_sums(sums, n_sums)) return hipErrorInvalidValue;
  F32Args wide[kMaxWgrads], narrow[kMaxWgrads];
  int n_wide = 0, n_narrow = 0;
  for (int i = 0; i < n; ++i) {
    const WgradItem& w = items[i];
    if (!gemm_f32_supported(2, w.M, w.N, K, w.dout, w.in, w.dw, GemmEpilogue())) return hipErrorInvalidValue;
    const F32Args a{(const float*)w.dout, (const float*)w.in, w.dw, w.M, w.N, K, nullptr, nullptr, nullptr, nullptr};
    if (use_wide(2, w.M, w.N, K)) wide[n_wide++] = a;
    else narrow[n_narrow++] = a;
  }
  hipError_t e = hipSuccess;
  // (the sums go with the last launch)
  if (n_wide > 0) e = launch_f32_group<2, 2, 1>(wide, n_wide, sums, n_narrow > 0 ? 0 : n_sums, st);
  if (e == hipSuccess && n_narrow > 0) e = launch_f32_group<1, 1, 4>(narrow, n_narrow, sums, n_sums, st);
  return e;
}

}  // namespace gpts

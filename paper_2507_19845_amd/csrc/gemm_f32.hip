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
// Two arrangements of the four waves:
//   2 x 2 x 1  a 64 x 64 tile of C, slices of 32 k
//   1 x 1 x 4  a 32 x 32 tile, slices of 64 k of which each wave multiplies a quarter; the four
//              partial tiles are added through LDS in fixed order.  Four times the workgroups, each
//              a quarter as long: the form for products that do not fill the chip.
// Slices travel global -> registers -> LDS, two slices ahead in registers and double buffered in
// LDS, one barrier per slice.
// Bound: the fp32 matrix pipe (157 TFLOP/s) where there are tiles enough, launch and memory
// latency below that.  Measured against gemm_simple_kernel (64 x 64 x 16, fp32 FMA), which served
// these products before: NT 4096x4096x4096 1911 -> 1137 us (121 TFLOP/s), 999x2048x512
// 53 -> 22 us, NN 999x512x2048 243 -> 28 us, TN 512x512x999 129 -> 11 us, NT 128x128x128
// 11.6 -> 7.4 us (launch bound).
#include "kernels.hpp"

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

// One operand's tile of R rows x BK k: global loads into registers, LDS stores, fragment reads.
template <int R, int BK, bool KMAJOR> struct F32Operand {
  static constexpr int PER = R * BK / 4 / 256;              // 16-byte pieces per thread
  static constexpr int CPR = KMAJOR ? R / 4 : BK / 4;       // pieces per row of the LDS tile
  // K-major rows are padded by 8 floats so that the four k-rows a wave reads together lie 32
  // banks apart; K-contiguous rows are swizzled instead (below)
  static constexpr int PITCH = KMAJOR ? R + 8 : BK;
  static constexpr int FLOATS = (KMAJOR ? BK : R) * PITCH;
  static_assert(R * BK / 4 % 256 == 0, "whole pieces per thread");

  const float* src[PER];   // this thread's pieces in slice 0
  int k_of[PER];           // their first k
  int dst[PER];            // LDS offsets (floats)

  __device__ __forceinline__ void init(const float* X, int r0, int rtotal, int K) {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int idx = threadIdx.x + 256 * p, row = idx / CPR, c = idx % CPR;
      if constexpr (KMAJOR) {
        const int col = r0 + c * 4 < rtotal ? r0 + c * 4 : 0;   // past the edge: any valid column
        src[p] = X + (size_t)row * rtotal + col;
        k_of[p] = row;
        dst[p] = row * PITCH + c * 4;
      } else {
        const int gr = r0 + row < rtotal ? r0 + row : rtotal - 1;
        src[p] = X + (size_t)gr * K + c * 4;
        k_of[p] = c * 4;
        // a wave reads the rows 2i + b (i = 0..15) at one piece: XOR with i spreads them
        dst[p] = row * PITCH + (c ^ ((row >> 1) & 7)) * 4;
      }
    }
  }
  // pieces of slice kt; k past the end of the contraction reads as zero (both operands do, so
  // nothing is multiplied by what lies there)
  __device__ __forceinline__ void load(f32x4 (&v)[PER], int kt, int rtotal, int K) const {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      const size_t step = KMAJOR ? (size_t)kt * BK * rtotal : (size_t)kt * BK;
      v[p] = kt * BK + k_of[p] < K ? *reinterpret_cast<const f32x4*>(src[p] + step) : zero;
    }
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
        const f32x4 v = *reinterpret_cast<const f32x4*>(tile + row * PITCH + (((k0 >> 2) + g) ^ ((row >> 1) & 7)) * 4);
#pragma unroll
        for (int s = 0; s < 4; ++s) f[b][s] = v[s];
      }
    }
  }
};

template <int EPI> __device__ __forceinline__ void f32_store4(const F32Args& a, int m, int n, f32x4 v) {
  if (m >= a.M || n >= a.N) return;
  const size_t o = (size_t)m * a.N + n;
  auto ld4 = [](const float* p) { return *reinterpret_cast<const f32x4*>(p); };
  if constexpr (EPI == F32_ACCUM) {
    *reinterpret_cast<f32x4*>(a.C + o) = ld4(a.C + o) + v;
  } else {
    if (a.bias) v += ld4(a.bias + n);
    if constexpr (EPI == F32_GELU_TANH || EPI == F32_GELU_ERF) {
      f32x4 gq;
#pragma unroll
      for (int e = 0; e < 4; ++e) gq[e] = gelu_f<EPI == F32_GELU_TANH ? 0 : 1>(v[e]);
      *reinterpret_cast<f32x4*>(a.C + o) = v;
      *reinterpret_cast<f32x4*>(a.gelu_out + o) = gq;
    } else {
      if constexpr (EPI == F32_DGELU_TANH || EPI == F32_DGELU_ERF) {
        const f32x4 u = ld4(a.dgelu_u + o);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] *= gelu_grad_f<EPI == F32_DGELU_TANH ? 0 : 1>(u[e]);
      }
      if (a.residual) v += ld4(a.residual + o);
      *reinterpret_cast<f32x4*>(a.C + o) = v;
    }
  }
}

// floats of LDS a tile's two stages take
template <int WM, int WN, int WK, bool A_KM, bool B_KM> constexpr int f32_lds_floats() {
  constexpr int BK = WK == 1 ? 32 : 64;
  return 2 * (F32Operand<32 * WM, BK, A_KM>::FLOATS + F32Operand<32 * WN, BK, B_KM>::FLOATS);
}
template <int WM, int WN, int WK, bool A_KM, bool B_KM, int EPI>
__device__ __forceinline__ void f32_tile(const F32Args& a, int tile_m, int tile_n, float* const lds) {
  static_assert(WM * WN * WK == 4 && (WK == 1 || (WM == 1 && WN == 1)), "four waves; a split contraction has one tile");
  constexpr int BM = 32 * WM, BN = 32 * WN, BK = WK == 1 ? 32 : 64, KW = BK / WK;
  using OpA = F32Operand<BM, BK, A_KM>;
  using OpB = F32Operand<BN, BK, B_KM>;
  constexpr int STAGE = OpA::FLOATS + OpB::FLOATS;
  static_assert(2 * STAGE >= 4 * 4 * 256, "the four partial tiles fit");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  OpA opA;
  OpB opB;
  opA.init(a.A, m0, a.M, a.K);
  opB.init(a.B, n0, a.N, a.K);
  const int nk = (a.K + BK - 1) / BK;

  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 ra[2][OpA::PER], rb[2][OpB::PER];
  auto load = [&](int t, int r) {
    if (t < nk) {
      opA.load(ra[r], t, a.M, a.K);
      opB.load(rb[r], t, a.N, a.K);
    }
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
  load(0, 0);
  load(1, 1);
  opA.store(ra[0], lds);
  opB.store(rb[0], lds + OpA::FLOATS);
  load(2, 0);
  __syncthreads();
  for (int t = 0; t < nk; t += 2) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // slice t+h lies in stage h; the registers [h^1] hold slice t+h+1, which goes to the other
      // stage (every wave left that one before the last barrier)
      if (t + h < nk) {
        multiply(lds + h * STAGE);
        if (t + h + 1 < nk) {
          float* nxt = lds + (h ^ 1) * STAGE;
          opA.store(ra[h ^ 1], nxt);
          opB.store(rb[h ^ 1], nxt + OpA::FLOATS);
          load(t + h + 3, h ^ 1);
        }
        __syncthreads();
      }
    }
  }

  // acc[ib][jb][r] = C[2i + ib][2(4g + r) + jb] of the wave's block: columns 8g .. 8g+7 of a row
  const int i = lane & 15, g = lane >> 4;
  auto half = [&](int ib, int h) {
    return f32x4{acc[ib][0][2 * h], acc[ib][1][2 * h], acc[ib][0][2 * h + 1], acc[ib][1][2 * h + 1]};
  };
  if constexpr (WK == 1) {
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int h = 0; h < 2; ++h) f32_store4<EPI>(a, m0 + wm * 32 + 2 * i + ib, n0 + wn * 32 + 8 * g + 4 * h, half(ib, h));
  } else {
    // each wave adds up and stores one quarter of the tile (the loop's last barrier has freed the LDS)
    f32x4* part = reinterpret_cast<f32x4*>(lds);
#pragma unroll
    for (int q = 0; q < 4; ++q) part[(wave * 4 + q) * 64 + lane] = half(q >> 1, q & 1);
    __syncthreads();
    f32x4 v = part[wave * 64 + lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) v += part[(w * 4 + wave) * 64 + lane];
    f32_store4<EPI>(a, m0 + 2 * i + (wave >> 1), n0 + 8 * g + 4 * (wave & 1), v);
  }
}

template <int WM, int WN, int WK, bool A_KM, bool B_KM, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const F32Args a) {
  __shared__ __attribute__((aligned(16))) float lds[f32_lds_floats<WM, WN, WK, A_KM, B_KM>()];
  f32_tile<WM, WN, WK, A_KM, B_KM, EPI>(a, blockIdx.y, blockIdx.x, lds);
}
// Several weight gradients in one launch.
struct F32Group {
  F32Args p[kMaxWgrads];
  int first[kMaxWgrads];   // first workgroup of a product
};
template <int WM, int WN, int WK> __global__ __launch_bounds__(256) void gemm_f32_group_kernel(const F32Group g) {
  __shared__ __attribute__((aligned(16))) float lds[f32_lds_floats<WM, WN, WK, true, true>()];
  int k = 0;
#pragma unroll
  for (int i = 1; i < kMaxWgrads; ++i)
    if ((int)blockIdx.x >= g.first[i]) k = i;
  const int id = blockIdx.x - g.first[k], tiles_n = (g.p[k].N + 32 * WN - 1) / (32 * WN);
  f32_tile<WM, WN, WK, true, true, F32_ACCUM>(g.p[k], id / tiles_n, id % tiles_n, lds);
}

// 64 x 64 tiles where there are at least 320 of them, else 32 x 32 tiles with a split contraction.
// Measured (64 / 32): 512 tiles (NT 999x2048x512) 22.3 / 25.6 us; 384 tiles (NT 999x1536x512)
// 22.9 / 22.9; 256 tiles, one per CU and none to hide its latency (TN 2048x512x999) 29.7 / 27.1;
// 192 tiles (TN 1536x512x999) 29.4 / 21.8; 128 tiles (NN 999x512x2048) 51.9 / 27.7.
bool use_wide(int M, int N) { return (long)((M + 63) / 64) * ((N + 63) / 64) >= 320; }

template <bool A_KM, bool B_KM, int EPI> hipError_t launch_f32(const F32Args& a, hipStream_t st) {
  if (use_wide(a.M, a.N)) {
    hipLaunchKernelGGL((gemm_f32_kernel<2, 2, 1, A_KM, B_KM, EPI>), dim3((a.N + 63) / 64, (a.M + 63) / 64), dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL((gemm_f32_kernel<1, 1, 4, A_KM, B_KM, EPI>), dim3((a.N + 31) / 32, (a.M + 31) / 32), dim3(256), 0, st, a);
  }
  return hipGetLastError();
}

template <int WM, int WN, int WK> hipError_t launch_f32_group(const F32Args* a, int n, hipStream_t st) {
  F32Group g;
  int blocks = 0;
  for (int i = 0; i < kMaxWgrads; ++i) {
    g.p[i] = a[i < n ? i : 0];
    g.first[i] = i < n ? blocks : 0x7fffffff;      // (never reached)
    if (i < n) blocks += ((a[i].M + 32 * WM - 1) / (32 * WM)) * ((a[i].N + 32 * WN - 1) / (32 * WN));
  }
  hipLaunchKernelGGL((gemm_f32_group_kernel<WM, WN, WK>), dim3(blocks), dim3(256), 0, st, g);
  return hipGetLastError();
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

// 16-byte pieces: every contiguous dimension a multiple of 4, every pointer 16-byte aligned; the
// grid's y dimension holds at most 65535 tile rows.
bool gemm_f32_supported(int form, int M, int N, int K, const void* A, const void* B, const void* C,
                        const GemmEpilogue& ep) {
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
hipError_t gemm_f32_wgrad_group(const WgradItem* items, int n, int K, hipStream_t st) {
  if (n < 1 || n > kMaxWgrads) return hipErrorInvalidValue;
  F32Args wide[kMaxWgrads], narrow[kMaxWgrads];
  int n_wide = 0, n_narrow = 0;
  for (int i = 0; i < n; ++i) {
    const WgradItem& w = items[i];
    if (!gemm_f32_supported(2, w.M, w.N, K, w.dout, w.in, w.dw, GemmEpilogue())) return hipErrorInvalidValue;
    const F32Args a{(const float*)w.dout, (const float*)w.in, w.dw, w.M, w.N, K, nullptr, nullptr, nullptr, nullptr};
    if (use_wide(w.M, w.N)) wide[n_wide++] = a;
    else narrow[n_narrow++] = a;
  }
  hipError_t e = hipSuccess;
  if (n_wide > 0) e = launch_f32_group<2, 2, 1>(wide, n_wide, st);
  if (e == hipSuccess && n_narrow > 0) e = launch_f32_group<1, 1, 4>(narrow, n_narrow, st);
  return e;
}

}  // namespace gpts

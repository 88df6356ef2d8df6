// bf16 (and, for the forward phase of cfg.fwd_fp16 stages, fp16) matrix products on the gfx950
// matrix cores: which tile of gemm_mi16_kernel (gemm_tiles.hpp) a product runs on, and the tiled
// weight images.
#include "gemm_tiles.hpp"

namespace gpts {
namespace {

// ---- operand images -----------------------------------------------------------------
// image[tile of 256 rows][slice of 64][slot] with slot = row*8 + physical chunk, holding logical
// chunk (physical ^ swizzle(row)) of weight row tile*256+row, k = slice*64 + chunk*8 .. +7.  Rows
// past N are zero.  One workgroup per (slice, tile): reads and writes are whole 128-byte rows whose
// 16-byte chunks change places, nothing is staged.  A rest of K below 64 is left out: products of
// such a length do not read images.
// TO_F16: the image holds the values converted to fp16 (exact for magnitudes in
// [2^-14, 65504]; smaller ones become fp16 subnormals, absolute error <= 2^-25; larger ones
// saturate), for products whose other operand is an fp16 activation.
template <bool TO_F16>
__global__ __launch_bounds__(256) void prepare_image_kernel(const bf16* __restrict__ src, bf16* __restrict__ img,
                                                            int N, int K) {
  constexpr int PER = 256 * (kImageK / 8) / 256;
  const int kt = blockIdx.x, tn = blockIdx.y, nk = K / kImageK;
  bf16* out = img + ((size_t)tn * nk + kt) * (256 * kImageK);
  bf16x8 v[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int slot = p * 256 + threadIdx.x, r = slot >> 3, c = (slot & 7) ^ swz_kc(r);
    if (tn * 256 + r < N) v[p] = *reinterpret_cast<const bf16x8*>(src + (size_t)(tn * 256 + r) * K + kt * kImageK + c * 8);
    else for (int e = 0; e < 8; ++e) v[p][e] = (bf16)0.f;
  }
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    bf16* dst = out + (size_t)(p * 256 + threadIdx.x) * 8;
    if constexpr (TO_F16) {
      f16x8 h;
#pragma unroll
      for (int e = 0; e < 8; ++e) h[e] = sat_f16((float)v[p][e]);
      *reinterpret_cast<f16x8*>(dst) = h;
    } else {
      *reinterpret_cast<bf16x8*>(dst) = v[p];
    }
  }
}

// ---- which tile ------------------------------------------------------------------------
// The tile whose estimated time is least: the fullest compute unit works ceil(tiles / 256) tiles one
// after the other, each ceil(K / 64) * slice + fixed microseconds.  The two numbers of a tile are
// fitted to measured products that fill whole rounds (random bf16 operands from HBM, M, N in
// 384 ... 20480, K in 320 ... 16384; the estimate is within 10 % of those); `fixed` is the first slice's
// arrival and the epilogue, which reads and writes fp32 in the weight gradients.  The line knows no
// costlier epilogue beyond 768 k (below), and takes 128x128 and 128x64 for lone workgroups of four stages also where
// they run with two (two_stages()).  Estimated | measured within steps, us: 4096x4096, K = 1024 in 256x256 30 | GeLU 46.9,
// GeLU' 51.6; 4096x3072, K = 1024 in 256x192 24 | 33.4; 2048x1536, K = 12288 in 128x128 82 | 121.
// What the choice is about: 2048x5120 is 160 tiles of 256x256 and 256 of 256x160 (K = 5120: 104 against
// 81 us), 2048x6144 is 192 and 256 of 256x192 (K = 12288: 279 against 266, weight gradient 253
// against 235 us), 4096x1024 is 64 and 256 of 128x128 (K = 4096: 76 against 30 us), 512x4096 is 256 of
// 128x64 (K = 1024: 8.0 us, 10.3 in 128x128), 512x1024 is 256 of 64x32 (K = 4096: 12 us, 25 in 128x128).
struct TileInfo {
  int bm, bn;
  float slice, fixed;         // NT and NN
  float slice_tn, fixed_tn;
};
constexpr TileInfo kTiles[N_TILES] = {
    {256, 256, 1.39f, 8.f, 1.45f, 21.4f},  {256, 192, 1.20f, 5.f, 1.17f, 17.f}, {256, 160, 0.95f, 4.5f, 0.98f, 14.f},
    {192, 192, 0.83f, 4.5f, 0.88f, 13.f}, {256, 128, 0.78f, 4.f, 0.66f, 11.f}, {128, 128, 0.40f, 5.f, 0.40f, 9.5f},
    {128, 64, 0.27f, 3.6f, 0.27f, 5.2f},  {64, 64, 0.17f, 2.6f, 0.18f, 3.3f},  {64, 32, 0.16f, 2.2f, 0.18f, 2.7f}};

// Weight gradients whose operands no longer stay in the 256 MB cache are not bound by the matrix pipe in
// every tile.  Each XCD reads a patch of 4 x 8 tiles, (4 bm + 8 bn) columns of a slice, and the eight
// together get 2.65 TB/s: 0.59 us a slice in 128x128.  6144x2048 (192 tiles of 256x256, 768 of 128x128):
// K = 10240, 168 MB of operands, 230 us in either; K = 14336, 235 MB, 316 against 344; K = 16384 355
// against 468; K = 32768 683 against 961.  2560x2560, K = 32768: 192x192 436, 128x128 614.
//
// Weight gradients in 256x128 and 128x128 share a unit in pairs (launch_wgrads()): beyond 256 tiles they go at the rate
// of kSharedTn a tile and unit, and a round that is not full costs a share (`lack`) of what is missing in it.  In step up to
// some 6000 k an XCD reads a patch of 4 x 16 of them for 64; beyond they drift apart and a slice takes an eighth longer.
// 256x256 | 256x128, us: 16384x4096, K = 2048 271 | 260, 4096 456 | 449, 8192 832 | 846, 32768 3137 | 3380; 6144x4096,
// K = 4096 200 | 165; 4096x4096, K = 512 33.5 | 38.8; layers of 4800 and 3456 tiles of 256x256, K = 2048 1285 | 1239
// and 931 | 880 (these two set `fixed_tn` of 256x256, too).
//
// Short contractions (short_contraction(), forward products and data gradients) are bound by their
// epilogues as much: they have numbers of their own, fitted to products of 64 ... 768 k (the estimate is
// within 8 % on average), a factor for what the epilogue does, and two forms with two stages, whose
// workgroups share a compute unit and need no whole rounds.  256x256 | 256x192 | 128x128 in two stages, us:
// 7784x9152, K = 256, GeLU' 122 | 135 | 101; 14608x13952, K = 128, bias 155 | 176 | 138; 32768x4096, K = 128,
// bias 98 | 117 | 98 and GeLU' 4096x2048, K = 512 31 | 28 | 19; 3560x1024, K = 64, GeLU' in 256x128, which the
// other estimate took, 13.4, in 64x64 8.7.
//
// A smaller tile has to promise 3 %, about what the estimates are good for.
struct ShortInfo { float start, slice, fixed; };
constexpr ShortInfo kShort[N_TILES] = {{-1.5f, 1.11f, 11.2f}, {-0.9f, 0.87f, 10.2f}, {-0.3f, 0.71f, 7.9f},
                                       {0.f, 0.67f, 7.9f},    {0.3f, 0.59f, 6.4f},   {0.8f, 0.36f, 3.9f},
                                       {1.3f, 0.26f, 2.4f},   {2.5f, 0.13f, 0.95f},  {2.5f, 0.11f, 0.54f}};
constexpr ShortInfo kShortShared128 = {2.75f, 0.37f, 1.87f}, kShortShared64 = {2.73f, 0.235f, 0.94f};
// what an epilogue moves and computes, over that of a bias or none: alone in a unit, sharing it
enum Cost { COST_PLAIN, COST_GELU, COST_DGELU, COST_RES32 };
constexpr float kCostAlone[] = {1.f, 1.55f, 1.75f, 1.5f}, kCostShared[] = {1.f, 1.8f, 2.f, 2.2f};

float short_us(Tile t, long tiles, long slices, Cost cost) {
  if (two_stages(tiles, slices * 64) && (t == TILE_128x128 || t == TILE_128x64)) {
    const ShortInfo& i = t == TILE_128x128 ? kShortShared128 : kShortShared64;
    return i.start + ((float)tiles / 256.f + 0.4f) * ((float)slices * i.slice + i.fixed * kCostShared[cost]);
  }
  const ShortInfo& i = kShort[t];
  return i.start + (float)((tiles + 255) / 256) * ((float)slices * i.slice + i.fixed * kCostAlone[cost]);
}

struct SharedInfo { float start, slice, fixed, lack; };
constexpr SharedInfo kSharedTn256x128 = {5.1f, 0.72f, 8.3f, 0.42f}, kSharedTn128x128 = {3.0f, 0.41f, 4.3f, 0.47f};
constexpr long kInStep = 6144;   // k
// of a weight gradient's tiles, more than 256 of them, whose operands hold so many bytes
float shared_tn_us(Tile t, long tiles, long K, float operand_bytes) {
  const SharedInfo& i = t == TILE_256x128 ? kSharedTn256x128 : kSharedTn128x128;
  const float patch = (float)((K <= kInStep ? 2 : 4) * kTiles[t].bm + 8 * kTiles[t].bn);
  float slice = K <= kInStep ? i.slice : 1.125f * i.slice;
  if (operand_bytes > 200e6f) slice = fmaxf(slice, patch * (64 * 2 * 8 / 2.65e6f));
  const float rounds = (float)tiles / 256.f;
  return i.start + (rounds + i.lack * (ceilf(rounds) - rounds)) * ((float)((K + 63) / 64) * slice + i.fixed);
}

struct Product { int M, N; };
// batch: products in one launch whose tile rows follow on
Tile choose_tile(int form, const Product* p, int n, long K, Cost cost, int batch = 1) {
  Tile best = TILE_256x256;
  float best_us = 0.f, operand_bytes = 0.f;
  for (int q = 0; q < n; ++q) operand_bytes += 2.f * (float)K * ((float)p[q].M + (float)p[q].N);
  for (int t = 0; t < N_TILES; ++t) {
    const TileInfo& i = kTiles[t];
    long tiles = 0;
    for (int q = 0; q < n; ++q) tiles += (long)batch * ((p[q].M + i.bm - 1) / i.bm) * ((p[q].N + i.bn - 1) / i.bn);
    const long rounds = (tiles + 255) / 256, slices = (K + 63) / 64;
    float slice = form == 2 ? i.slice_tn : i.slice, fixed = form == 2 ? i.fixed_tn : i.fixed;
    if (form == 2 && operand_bytes > 200e6f) slice = fmaxf(slice, (float)(4 * i.bm + 8 * i.bn) * (64 * 2 * 8 / 2.65e6f));
    float us = (float)rounds * ((float)slices * slice + fixed);
    if (form != 2 && short_contraction(K)) us = short_us((Tile)t, tiles, slices, cost);
    if (form == 2 && tiles > 256 && (t == TILE_256x128 || t == TILE_128x128)) us = shared_tn_us((Tile)t, tiles, K, operand_bytes);
    if (t == 0 || us < 0.97f * best_us) {
      best = (Tile)t;
      best_us = us;
    }
  }
  return best;
}
Tile choose_tile(int form, int M, int N, long K, Cost cost, int batch = 1) {
  const Product p{M, N};
  return choose_tile(form, &p, 1, K, cost, batch);
}

// Whether weight gradients in one launch gain on a launch each.  What they gain is the rounds that their
// partly filled last ones share.  What they lose is step: the workgroups of an XCD read each slice of an operand
// once from memory while they walk the contraction together, a new launch lines them up again, and in a long
// one the rounds drift apart (12 rounds of K = 32768: 35 GiB moved against 19.5).  So not with long contractions
// where under a sixteenth of the rounds is shared.  One launch | a launch each, us a layer, hidden and ffn:
//   4096, 16384, no shared round of 12   K = 12288 3557 | 3568   K = 16384 4696 | 4691   K = 32768 9590 | 9187
//   8192, 32768, none of 48              K = 4096  5304 | 5372   K = 16384 19723 | 18836
//   6144, 24576, one of 28               K = 8192  5558 | 5635   K = 24576 16542 | 16051
//   5120, 20480, two of 21               K = 32768 15602 | 16130     3072, 12288, two of 9  K = 49152 8427 | 8440
bool worth_one_launch(Tile t, const Product* p, int n, long K) {
  long apart = 0, tiles = 0;
  for (int q = 0; q < n; ++q) {
    const long own = (long)((p[q].M + kTiles[t].bm - 1) / kTiles[t].bm) * ((p[q].N + kTiles[t].bn - 1) / kTiles[t].bn);
    apart += (own + 255) / 256;
    tiles += own;
  }
  return K < 16384 || 16 * (apart - (tiles + 255) / 256) >= apart;
}

}  // namespace

bool gemm_mfma_supported(int form, int M, int N, int K) {
  (void)form;
  return M >= 64 && N >= 64 && K >= 64 && M % 8 == 0 && N % 8 == 0 && K % 64 == 0 &&
         (size_t)M * K < (1ull << 31) && (size_t)N * K < (1ull << 31);
}

// A weight-gradient product whose contraction is split over several buffers can run as one launch
// (K here is the length of one segment: whole slices, so no slice straddles two buffers): one fp32
// read-modify-write and one epilogue instead of one per micro-batch, and the four products of a layer in
// one launch where that gains (worth_one_launch()).  It changes the fp32 summation order over the
// tokens.  It is taken from four micro-batches on, and with two or three only for matrices of at least 100
// tiles of 256x256 with segments of whole 128 rows; other matrices keep the bits of the unsplit backward
// there.  That line is one of results and
// not of speed, one launch being the faster everywhere.  A layer's weight phase, a launch per micro-batch
// and matrix | one launch, us, 2 / 3 / 4 micro-batches:
//   hidden 320, 192 tokens   37 | 11    49 | 12    65 | 12      1024, 4096   305 | 242    461 | 353    613 | 466
//   hidden 1024, 512 tokens  81 | 42   119 | 52   154 | 61      4096, 4096  2769 | 2485  4118 | 3619  5508 | 4775
bool gemm_wgrad_segments_supported(int M, int N, int K, int segments) {
  if (!gemm_mfma_supported(2, M, N, K)) return false;
  return segments >= 4 || ((long)((M + 255) / 256) * ((N + 255) / 256) >= 100 && K % 128 == 0);
}

int gemm_mfma_colsum_rows(int M, int N, int K) {
  const int bm = kTiles[choose_tile(1, M, N, K, COST_DGELU)].bm;   // of the product with the GeLU' epilogue
  return 2 * ((M + bm - 1) / bm);
}

size_t gemm_image_elems(int N, int K) { return (size_t)((N + 255) / 256) * 256 * K; }

hipError_t gemm_prepare_image(const void* src, void* img, int N, int K, hipStream_t st, bool to_f16) {
  const dim3 g(K / kImageK, (N + 255) / 256);
  if (g.x == 0) return hipSuccess;
  if (to_f16)
    hipLaunchKernelGGL(prepare_image_kernel<true>, g, dim3(256), 0, st, (const bf16*)src, (bf16*)img, N, K);
  else
    hipLaunchKernelGGL(prepare_image_kernel<false>, g, dim3(256), 0, st, (const bf16*)src, (bf16*)img, N, K);
  return hipGetLastError();
}

bool gemm_fwd_f16_supported(int M, int N, int K) {
  return M >= 1 && N >= 8 && N % 8 == 0 && K >= 128 && K % 128 == 0 && (size_t)M * K < (1ull << 31) &&
         (size_t)((N + 255) / 256) * 256 * K < (1ull << 31);
}

namespace {
// MfmaArgs::once: from the 32 MB of the L2s on.  A smaller matrix may still be there from the call before, or be read
// from there by the next.  Cached | non-temporal, us a step.  Accumulated: 4096 tokens 1024 wide 2005 | 1986, 2048 tokens
// 5120 wide 7579 | 7457, 12288 wide in 12 heads 6342 | 6259, backward of 2048 tokens 2048 wide 1245 | 1215; 512 tokens 832
// wide (24 MB a layer) 123.8 | 125.5, 192 tokens 320 wide 298.7 | 299.9.  u on top: 4096 tokens 1024 wide 1997 | 1973, forward
// of 3968 tokens 2048 wide 888 | 882, 8 x 4096 tokens 4096 wide 141.9 | 141.2 ms.  u alone where the launch behind reads it again:
// recompute == 1, backward of 2048 tokens 2048 wide 1241 | 1241, 4096 tokens 1024 wide 1050 | 1047, 8192 tokens 512 wide 928 |
// 919, 4096 tokens 4096 wide 4854 | 4874; recompute == 2, the same 1533 | 1521, 1247 | 1219, 1104 | 1085, 5812 | 5804, 2048 tokens
// 5120 wide 4546 | 4552; fp16, 2048 tokens 2048 wide 962 | 962 (two runs differ by 0.5 %, the 4096-wide by 1.4).
constexpr size_t kOnceBytes = (size_t)32 << 20;
MfmaArgs make_args(int M, int N, int K, const void* A, const void* B, void* C, const GemmEpilogue& ep) {
  MfmaArgs a;
  a.A = (const bf16*)A; a.B = (const bf16*)B; a.C = C;
  a.M = M; a.N = N; a.K = K;
  a.bias = (const bf16*)ep.bias; a.residual = ep.residual;
  a.gelu_out = (bf16*)ep.gelu_out; a.dgelu_u = (const bf16*)ep.dgelu_u;
  a.colsum = ep.dgelu_u ? ep.colsum_partial : nullptr;
  a.once = (ep.gelu_out || ep.dgelu_u) && (size_t)2 * ep.batch * M * N >= kOnceBytes;
  return a;
}
int fwd_epilogue(const GemmEpilogue& ep) {
  if (ep.gelu_out) return ep.gelu_kind == 0 ? EPI_GELU_TANH : EPI_GELU_ERF;
  if (ep.residual && ep.residual_f32) return ep.out_f32 ? EPI_BIAS_RES32_OUT32 : EPI_BIAS_RES32_OUT16;
  return ep.residual ? EPI_BIAS_RES : EPI_BIAS;
}
Cost cost_of(const GemmEpilogue& ep) {
  if (ep.gelu_out) return COST_GELU;
  if (ep.dgelu_u) return COST_DGELU;
  return ep.residual && ep.residual_f32 ? COST_RES32 : COST_PLAIN;
}
}  // namespace

hipError_t gemm_fwd_f16(int M, int N, int K, const void* A, const void* b_image, void* C,
                        const GemmEpilogue& ep, hipStream_t st) {
  if (!gemm_fwd_f16_supported(M, N, K) || !b_image) return hipErrorInvalidValue;
  MfmaArgs a = make_args(M, N, K, A, b_image, C, ep);
  a.b_img = 1;
  return launch_gemm_fwd_f16(choose_tile(0, M, N, K, cost_of(ep)), fwd_epilogue(ep), a, st);
}

hipError_t gemm_mfma(int form, int M, int N, int K, const void* A, const void* B, void* C,
                     const GemmEpilogue& ep, hipStream_t st) {
  if (!gemm_mfma_supported(form, M, N, K)) return hipErrorInvalidValue;   // (whole slices of K only)
  if (form == 2) {
    const WgradItem w{M, N, A, B, (float*)C};
    return gemm_wgrad_group(&w, 1, K, ep.k_segments, ep.seg_stride_a, ep.seg_stride_b, st);
  }
  MfmaArgs a = make_args(M, N, K, A, B, C, ep);
  if (ep.batch < 1 || ep.batch > kMaxWindow || !window_stride_ok(ep.stride_r)) return hipErrorInvalidValue;
  a.batch = ep.batch;
  a.stride_a = ep.stride_a;
  a.stride_b = ep.stride_c;
  a.stride_r = (uint32_t)(ep.stride_r / 16);
  // (the order in which the rows of a column are summed is the tile's: a product that leaves column sums keeps it)
  const Tile t = choose_tile(form, M, N, K, cost_of(ep), a.colsum ? 1 : ep.batch);
  if (form == 1)
    return launch_gemm_dgrad(t, !ep.dgelu_u ? EPI_PLAIN : (ep.gelu_kind == 0 ? EPI_DGELU_TANH : EPI_DGELU_ERF), a, st);
  if (ep.b_image) {
    a.B = (const bf16*)ep.b_image;
    a.b_img = 1;
  }
  return launch_gemm_fwd(t, fwd_epilogue(ep), a, st);
}

hipError_t gemm_wgrad_group(const WgradItem* items, int n, int K, int segments, size_t seg_stride_dout,
                            size_t seg_stride_in, hipStream_t st, const ReduceSeg* sums, int n_sums) {
  if (n < 1 || n > kMaxWgrads || !few_sums(sums, n_sums)) return hipErrorInvalidValue;
  MfmaArgs a[kMaxWgrads];
  Product p[kMaxWgrads];
  size_t matrices = 0;   // bytes
  for (int i = 0; i < n; ++i) {
    const WgradItem& w = items[i];
    if (segments > 1 ? !gemm_wgrad_segments_supported(w.M, w.N, K, segments) : !gemm_mfma_supported(2, w.M, w.N, K))
      return hipErrorInvalidValue;
    a[i] = make_args(w.M, w.N, K, w.dout, w.in, w.dw, GemmEpilogue());
    a[i].batch = segments;
    a[i].stride_a = seg_stride_dout;
    a[i].stride_b = seg_stride_in;
    p[i] = Product{w.M, w.N};
    matrices += sizeof(float) * w.M * w.N;
  }
  for (int i = 0; i < n; ++i) a[i].once = matrices >= kOnceBytes;
  const long k_all = (long)K * segments;
  const Tile t = choose_tile(2, p, n, k_all, COST_PLAIN);
  if (n == 1 || worth_one_launch(t, p, n, k_all)) return launch_gemm_wgrad(t, a, n, sums, n_sums, st);
  for (int i = 0; i < n; ++i) {
    const hipError_t e = launch_gemm_wgrad(choose_tile(2, p + i, 1, k_all, COST_PLAIN), a + i, 1, nullptr, 0, st);
    if (e != hipSuccess) return e;
  }
  return n_sums == 0 ? hipSuccess : reduce_partials(sums, n_sums, st);
}

}  // namespace gpts

// C ABI of the library (see include/hidet_mi355x.h): argument validation, choice of the tile
// configuration, the tuner that enumerates the hardware-centric schedule space, and the launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/hidet_mi355x.h"
#include "registry.hpp"

namespace hidet {  // conv_patch.hip
hipError_t launch_conv_patch_f16(const GemmParams& p, int bm, hipStream_t stream);
hipError_t launch_conv_patch_bf16(const GemmParams& p, int bm, hipStream_t stream);
}  // namespace hidet

using namespace hidet;

// ------------------------------------------------------------------------------------------------
// Table of contents of the schedule space + the launchers registered by the instance objects.
// ------------------------------------------------------------------------------------------------
#define HIDET_ALL
static constexpr ConfigRow kConfigs[] = {
#define X16(idx, BM, BN, BK, WM, WN, MI, TA, SC) {idx, BM, BN, BK, WM, WN, MI, TA, SC, 0},
#define X32(idx, BM, BN, BK, WM, WN, MI, TA, SC) {idx, BM, BN, BK, WM, WN, MI, TA, SC, 1},
#include "configs.def"
#undef X16
#undef X32
};
static const int kNumConfigs = (int)(sizeof(kConfigs) / sizeof(kConfigs[0]));

// weak: a development build may leave some (configuration, type) objects out; their table slots stay empty
#define X16(idx, BM, BN, BK, WM, WN, MI, TA, SC)                                  \
  extern "C" void hidet_register_##idx##_1(Registry*) __attribute__((weak));    \
  extern "C" void hidet_register_##idx##_2(Registry*) __attribute__((weak));
#define X32(idx, BM, BN, BK, WM, WN, MI, TA, SC) extern "C" void hidet_register_##idx##_0(Registry*) __attribute__((weak));
#include "configs.def"
#undef X16
#undef X32

static const Registry& registry() {
  static Registry* r = [] {
    Registry* reg = new Registry();
    std::memset(reg, 0, sizeof(Registry));
#define X16(idx, BM, BN, BK, WM, WN, MI, TA, SC)                \
  if (hidet_register_##idx##_1) hidet_register_##idx##_1(reg); \
  if (hidet_register_##idx##_2) hidet_register_##idx##_2(reg);
#define X32(idx, BM, BN, BK, WM, WN, MI, TA, SC) \
  if (hidet_register_##idx##_0) hidet_register_##idx##_0(reg);
#include "configs.def"
#undef X16
#undef X32
    return reg;
  }();
  return *r;
}
#undef HIDET_ALL

static_assert(sizeof(kConfigs) / sizeof(kConfigs[0]) <= kMaxConfigs, "raise kMaxConfigs");
static constexpr bool tile_extents_are_powers_of_two() {
  for (const ConfigRow& r : kConfigs)
    if ((r.bm & (r.bm - 1)) != 0 || (r.bn & (r.bn - 1)) != 0) return false;
  return true;
}
static_assert(tile_extents_are_powers_of_two(), "the size-based choice shifts by the logarithm of a tile extent");

// ------------------------------------------------------------------------------------------------
// Problem description shared by GEMM, batched GEMM and conv.
// ------------------------------------------------------------------------------------------------
namespace {

struct Problem {
  int op = 0;  // 0 gemm (batched), 1 conv
  int dtype = 0;      // input type
  int wide_out = 0;   // 1: 16-bit inputs, fp32 output (and fp32 bias / residual)
  int transA = 0, transB = 0;
  long long batch = 1;
  int elem_mode = 0;  // 1: some operand is not 16-byte aligned -> element loads
  int packed = 0;     // convolution only: 1 = weights repacked to the tap-major K order (kh, kw, ic)
  int images = 0;     // convolution only: 1 = 1x1, its columns run through all images, ring schedule
  GemmParams p{};
  // conv-only key fields
  long long Nb = 0, OC = 0;
};

int elem_size(int dtype) { return dtype == HIDET_F32 ? 4 : 2; }
bool aligned(const void* ptr, size_t a) { return (reinterpret_cast<uintptr_t>(ptr) % a) == 0; }
constexpr long long kIntMax = 2147483647LL;
// Largest extent of a GEMM dimension (and of the input tensor of a convolution, in elements): the kernels keep
// such indices in 32 bits and step past them by at most one tile (or one gather window) before comparing.
constexpr long long kMaxDim = kIntMax - 65536;
// An operand spans (rows - 1) * ld + cols elements per batch entry and batch * stride over the batch; both are
// kept below 2^47 (no allocation is larger), so that neither the checks here nor the 64-bit offsets of the kernels
// can overflow.
constexpr long long kMaxExtent = 1LL << 47;
bool extent_ok(long long rows, long long ld, long long batch, long long stride) {
  if (ld > kMaxExtent || stride > kMaxExtent) return false;
  if (rows > 1 && ld > kMaxExtent / rows) return false;
  if (batch > 1 && stride > kMaxExtent / batch) return false;
  return true;
}
// a * b, saturating at 2^62 (a, b >= 0)
long long sat_mul(long long a, long long b) {
  constexpr long long lim = 1LL << 62;
  if (a == 0 || b == 0) return 0;
  return a > lim / b ? lim : a * b;
}

// GEMM: the output has the input type, or is fp32 for 16-bit inputs.  Convolution: same type only.
hidet_status_t check_dtypes(int in, int out, bool conv) {
  if (in < 0 || in > 2 || out < 0 || out > 2) return HIDET_ERR_INVALID_ARG;
  if (in != out && (conv || out != HIDET_F32)) return HIDET_ERR_UNSUPPORTED;
  return HIDET_OK;
}

hidet_status_t check_epilogue(const hidet_epilogue_t* epi, int dtype, bool conv) {
  if (!epi) return HIDET_OK;
  if (epi->struct_size != sizeof(hidet_epilogue_t)) return HIDET_ERR_INVALID_ARG;
  if (epi->bias_axis < 0 || epi->bias_axis > 2 || epi->act < 0 || epi->act > 1) return HIDET_ERR_INVALID_ARG;
  if (epi->bias_axis != HIDET_BIAS_NONE && !epi->bias) return HIDET_ERR_INVALID_ARG;
  if (conv && epi->bias_axis == HIDET_BIAS_PER_COL) return HIDET_ERR_INVALID_ARG;
  if (epi->out_map < 0 || epi->out_map > 1 || epi->prologue < 0 || epi->prologue > 1) return HIDET_ERR_INVALID_ARG;
  if (conv && epi->out_map != HIDET_MAP_PLAIN) return HIDET_ERR_INVALID_ARG;
  const size_t es = (size_t)elem_size(dtype);
  if (epi->bias_axis != HIDET_BIAS_NONE && !aligned(epi->bias, es)) return HIDET_ERR_ALIGNMENT;
  if (epi->residual && !aligned(epi->residual, es)) return HIDET_ERR_ALIGNMENT;
  if (!(epi->alpha == epi->alpha)) return HIDET_ERR_INVALID_ARG;  // NaN scale
  return HIDET_OK;
}

void fill_epilogue(GemmParams& p, const hidet_epilogue_t* epi) {
  p.alpha = 1.0f;
  p.bias = nullptr;
  p.bias_axis = 0;
  p.residual = nullptr;
  p.ldr = 0;
  p.strideR = 0;
  p.relu = 0;
  p.relu_a = p.relu_b = 0;
  p.out_map = 0;
  p.map_seq = p.map_d = p.map_heads = 1;
  p.d_seq = p.d_hd = make_fastdiv(1);
  if (epi) {
    p.alpha = epi->alpha;
    p.bias_axis = epi->bias_axis;
    p.bias = epi->bias_axis ? epi->bias : nullptr;
    p.residual = epi->residual;
    p.ldr = epi->ld_residual;
    p.strideR = epi->batch_stride_residual;
    p.relu = epi->act == HIDET_ACT_RELU;
    p.relu_a = epi->prologue == HIDET_PROLOGUE_RELU;  // the activation operand of a GEMM (make_conv_problem moves it to x)
  }
}

hidet_status_t make_gemm_problem(Problem& pr, int in, int out, int transA, int transB, long long batch, long long M,
                                 long long N, long long K, const void* A, long long lda, long long strideA,
                                 const void* B, long long ldb, long long strideB, void* C, long long ldc,
                                 long long strideC, const hidet_epilogue_t* epi) {
  hidet_status_t st = check_dtypes(in, out, false);
  if (st != HIDET_OK) return st;
  if (batch < 0 || M < 0 || N < 0 || K < 0) return HIDET_ERR_INVALID_ARG;
  if (M > kMaxDim || N > kMaxDim || K > kMaxDim || batch > kIntMax) return HIDET_ERR_UNSUPPORTED;
  const bool empty = (batch == 0 || M == 0 || N == 0);
  st = check_epilogue(epi, out, false);
  if (st != HIDET_OK) return st;
  if (!empty) {
    if (!C) return HIDET_ERR_INVALID_ARG;
    if (K > 0 && (!A || !B)) return HIDET_ERR_INVALID_ARG;
    if (lda < (transA ? M : K) || ldb < (transB ? K : N) || ldc < N) return HIDET_ERR_INVALID_ARG;
    if (strideA < 0 || strideB < 0 || strideC < 0) return HIDET_ERR_INVALID_ARG;
    if (!extent_ok(transA ? K : M, lda, batch, strideA) || !extent_ok(transB ? N : K, ldb, batch, strideB) ||
        !extent_ok(M, ldc, batch, strideC))
      return HIDET_ERR_UNSUPPORTED;
    if (batch > 1 && strideC < (M - 1) * ldc + N) return HIDET_ERR_INVALID_ARG;
    const bool head_split = epi && epi->out_map == HIDET_MAP_HEAD_SPLIT;
    if (head_split) {
      if (batch != 1) return HIDET_ERR_UNSUPPORTED;
      if (epi->map_seq <= 0 || epi->map_head_dim <= 0 || M % epi->map_seq != 0 || N % epi->map_head_dim != 0)
        return HIDET_ERR_INVALID_ARG;
    }
    if (epi && epi->residual && !head_split) {
      if (epi->ld_residual < N) return HIDET_ERR_INVALID_ARG;
      if (epi->batch_stride_residual < 0) return HIDET_ERR_INVALID_ARG;
      if (!extent_ok(M, epi->ld_residual, batch, epi->batch_stride_residual)) return HIDET_ERR_UNSUPPORTED;
    }
    const size_t es = (size_t)elem_size(in);
    if (!aligned(A, es) || !aligned(B, es) || !aligned(C, (size_t)elem_size(out))) return HIDET_ERR_ALIGNMENT;
  }
  pr.op = 0;
  pr.dtype = in;
  pr.wide_out = (in != out) ? 1 : 0;
  pr.transA = transA ? 1 : 0;
  pr.transB = transB ? 1 : 0;
  pr.batch = batch;
  GemmParams& p = pr.p;
  p.A = A;
  p.B = B;
  p.C = C;
  p.M = (int)M;
  p.N = (int)N;
  p.K = (int)K;
  p.lda = lda;
  p.ldb = ldb;
  p.ldc = ldc;
  p.strideA = strideA;
  p.strideB = strideB;
  p.strideC = strideC;
  fill_epilogue(p, epi);
  const int vec = 16 / elem_size(in);
  // vector loads need 16-byte aligned rows, no chunk straddling a matrix edge, and 32-bit in-tile offsets
  const long long a_contig = transA ? M : K, b_contig = transB ? K : N;
  const bool a_vec = aligned(A, 16) && lda % vec == 0 && strideA % vec == 0 && a_contig % vec == 0 && lda <= kMaxVecLd;
  const bool b_vec = aligned(B, 16) && ldb % vec == 0 && strideB % vec == 0 && b_contig % vec == 0 && ldb <= kMaxVecLd;
  pr.elem_mode = (a_vec && b_vec) ? 0 : 1;
  const size_t va = 4 * (size_t)elem_size(out);
  bool vs = aligned(C, va) && ldc % 4 == 0 && strideC % 4 == 0;
  if (p.residual) vs = vs && aligned(p.residual, va) && p.ldr % 4 == 0 && p.strideR % 4 == 0;
  bool contiguous4 = true;  // row-major: four consecutive columns of a row are always adjacent
  if (!empty && epi && epi->out_map == HIDET_MAP_HEAD_SPLIT) {
    p.out_map = 1;
    p.map_seq = (int)epi->map_seq;
    p.map_d = (int)epi->map_head_dim;
    p.map_heads = (int)(N / epi->map_head_dim);
    p.d_seq = make_fastdiv(epi->map_seq);
    p.d_hd = make_fastdiv(epi->map_head_dim);
    contiguous4 = epi->map_head_dim % 4 == 0;
    vs = contiguous4 && aligned(C, va) && (!p.residual || aligned(p.residual, va));
  }
  p.vec_store = vs ? 2 : (contiguous4 ? 1 : 0);
  // rows at least 4 KB apart: write the output through the L2 (see store_group)
  if (vs && p.out_map == 0 && elem_size(out) == 2 && p.ldc * 2 >= 4096) p.vec_store = 3;
  p.out_inner = 1;
  p.out_outer = 0;
  std::memset(&p.g, 0, sizeof(p.g));
  p.g.d_khw = p.g.d_kw = p.g.d_owp = p.g.d_oh = p.g.d_ic = make_fastdiv(1);
  return HIDET_OK;
}

hidet_status_t make_conv_problem(Problem& pr, int in, int out, long long Nb, long long IC, long long H, long long W,
                                 long long OC, long long KH, long long KW, long long sh, long long sw, long long ph,
                                 long long pw, const void* x, const void* w, void* y, const hidet_epilogue_t* epi) {
  hidet_status_t st = check_dtypes(in, out, true);
  if (st != HIDET_OK) return st;
  if (Nb < 0 || IC < 0 || H < 0 || W < 0 || OC < 0 || KH <= 0 || KW <= 0 || sh <= 0 || sw <= 0 || ph < 0 || pw < 0)
    return HIDET_ERR_INVALID_ARG;
  st = check_epilogue(epi, out, true);
  if (st != HIDET_OK) return st;
  // every factor is bounded before a product is formed (the products below then stay under 2^62)
  if (Nb > kMaxDim || IC > kMaxDim || OC > kMaxDim || H > 32767 || W > 32767 || KH > 32767 || KW > 32767 ||
      ph > 32767 || pw > 32767 || sh > 32767 || sw > 32767 || Nb * IC > kMaxDim)
    return HIDET_ERR_UNSUPPORTED;
  const long long OH = (H + 2 * ph - KH) >= 0 ? (H + 2 * ph - KH) / sh + 1 : 0;
  const long long OW = (W + 2 * pw - KW) >= 0 ? (W + 2 * pw - KW) / sw + 1 : 0;
  // GEMM columns enumerate output positions with every output row padded to a multiple of 8 (see ConvGeom)
  const long long OWP = (OW + 7) / 8 * 8;
  const long long M = OC, N = Nb * OH * OWP, K = IC * KH * KW;
  // the gather keeps input rows and columns (padding included) in signed 16-bit fields and element
  // offsets in 32 bits
  if (M > kMaxDim || N > kMaxDim || K > kMaxDim || Nb * IC * H * W > kMaxDim || H + 2 * ph > 32767 ||
      W + 2 * pw > 32767)
    return HIDET_ERR_UNSUPPORTED;
  const bool empty = (M == 0 || N == 0);
  if (!empty) {
    if (!y) return HIDET_ERR_INVALID_ARG;
    if (K > 0 && (!x || !w)) return HIDET_ERR_INVALID_ARG;
    const size_t es = (size_t)elem_size(in);
    if (!aligned(x, es) || !aligned(w, es) || !aligned(y, es)) return HIDET_ERR_ALIGNMENT;
  }
  pr.op = 1;
  pr.packed = 0;
  pr.dtype = in;
  pr.wide_out = 0;
  pr.transA = 0;
  pr.transB = 0;
  pr.batch = 1;
  pr.Nb = Nb;
  pr.OC = OC;
  GemmParams& p = pr.p;
  p.A = w;
  p.B = x;
  p.C = y;
  p.M = (int)M;
  p.N = (int)N;
  p.K = (int)K;
  p.lda = K;
  p.ldb = 0;
  p.ldc = 0;
  p.strideA = p.strideB = p.strideC = 0;
  fill_epilogue(p, epi);
  p.relu_b = p.relu_a;  // the activation operand of the convolution is x, the B operand of the implicit GEMM
  p.relu_a = 0;
  p.ldr = 0;
  p.strideR = 0;
  p.g = ConvGeom{(int)IC, (int)H, (int)W, (int)KH, (int)KW, (int)sh, (int)sw, (int)ph, (int)pw, (int)OH, (int)OW,
                 (int)OWP, (int)(Nb * IC * H * W), make_fastdiv(KH * KW), make_fastdiv(KW),
                 make_fastdiv(OWP > 0 ? OWP : 1), make_fastdiv(OH > 0 ? OH : 1), (int)(H * W),
                 make_fastdiv(IC > 0 ? IC : 1)};
  p.out_inner = OH * OW;
  p.out_outer = OC * OH * OW;
  const int vec = 16 / elem_size(in);
  pr.elem_mode = (aligned(w, 16) && K % vec == 0 && K <= kMaxVecLd) ? 0 : 1;
  const size_t va = 4 * (size_t)elem_size(out);
  // a group of four positions never leaves its (padded) output row, so it is always contiguous in y;
  // it is aligned to four elements when every output row is
  bool vs = aligned(y, va) && OW % 4 == 0;
  if (p.residual) vs = vs && aligned(p.residual, va);
  p.vec_store = vs ? 2 : 1;
  return HIDET_OK;
}

LaunchFn find_launcher(const Problem& pr, int config) {
  if (config < 0 || config >= kNumConfigs) return nullptr;
  // The ring schedule is built without the run-time output map; a head-split problem takes the same tile's
  // element-mode variant, whose launcher then picks the through-registers form of the schedule.
  if (pr.images != 0) return registry().fn[config][pr.dtype][kPointwiseVariant];
  // repacked weights: the K axis is (kh, kw, ic) and a K tile must lie within one filter tap
  if (pr.packed) return pr.p.g.IC % kConfigs[config].bk == 0 ? registry().fn[config][pr.dtype][kConvTapVariant] : nullptr;
  // The ring schedule is also built without the input prologue (its direct loads bypass the registers): such a
  // problem takes the through-registers form likewise.
  const int elem = ((pr.p.out_map != 0 || pr.p.relu_a != 0 || pr.p.relu_b != 0) && kConfigs[config].sched == 1) ? 1 : pr.elem_mode;
  const int variant = pr.op == 1 ? conv_variant(elem) : gemm_variant(pr.transA, pr.transB, elem);
  // fp32 output from 16-bit inputs: the kernels that the K-parallel form uses for its partial sums are ordinary
  // kernels with an fp32 output type
  return registry().fn[config][pr.dtype][(pr.wide_out ? kPartialVariants : 0) + variant];
}

// The fp32-output kernel of a configuration: writes the partial sums of the K-parallel form.
LaunchFn find_partial_launcher(const Problem& pr, int config) {
  if (config < 0 || config >= kNumConfigs) return nullptr;
  if (pr.packed)
    return pr.p.g.IC % kConfigs[config].bk == 0 ? registry().fn[config][pr.dtype][kConvTapVariant + 1] : nullptr;
  const int elem = ((pr.p.relu_a != 0 || pr.p.relu_b != 0) && kConfigs[config].sched == 1) ? 1 : pr.elem_mode;  // as in find_launcher
  const int variant = pr.op == 1 ? conv_variant(elem) : gemm_variant(pr.transA, pr.transB, elem);
  return registry().fn[config][pr.dtype][kPartialVariants + variant];
}

// Convolutions in 16-bit types on a long K.  A workgroup whose wave groups split K owns a compute unit, and its time
// hardly depends on its tile's neighbours: one round of them costs K times a rate of the tile (3x3, 512 channels,
// K = 4608: 16x16 11 us, 32x16 12, 32x32 18, 64x32 23, 64x64 36, 128x64 45, 128x128 67), a second round as much
// again.  So the smallest such tile whose workgroups are all resident at once is taken; measured against the choice
// below over batches 1 to 64 of 64x56x56, 128x28x28, 256x14x14 and 512x7x7, 3x3 and 5x5: 64 images of 512x7x7 69 -> 46 us,
// 256x14x14 44 -> 38 us, 6 images of 256x14x14 20 -> 13.5 us, one of 512x7x7 16 -> 11 us.  Large tiles have to be
// mostly output, not padding, and on a short K (fill and drain of the pipeline count) they need the round nearly full,
// or lose to small tiles that share a compute unit (128x28x28, 7 images, K = 1152: 64x64 18 us, 128x64 17 us, two
// 64x32 tiles of the two-stage form 15 us); the largest need half a round in any case (repacked weights allow only K tiles
// that divide IC: 5 images of 128x27x27, 5x5: 68 tiles of 128x64 33 us, 270 of 64x32 28 us).  On a long K the 64x64
// and 128x64 tiles may be half padding: what they compete with there are two-stage tiles (36 images of 512x13x13, 80
// channels, 3x3: 36 us on 234 of 64x64, 59 us on 351 two-stage tiles of 32x64).
// With strides above 2 the gather is one load per element, so the sixteen wavefronts of a K-splitting tile have more to win
// over the four of the others: they do so half padded, from K = 768 on, and the 64x32 tile (32x32 of at most 32 channels)
// also with one and a half workgroups per compute unit (40 images of 192x14x15, 512 channels, 3x3, stride 3: 34 us on 200
// tiles of 64x64, 46 us on 400 two-stage tiles of 64x32; 5 of 160x56x56, 512 channels, stride 4: 36 us on 280 tiles of
// 64x32, 42 us on 144 of 64x64, 47 us two-stage).  -1: none fits.
constexpr long long kConvLongK = 2048;
int one_round_config(const Problem& pr) {
  constexpr long long kComputeUnits = 256;
  const long long M = pr.p.M, N = pr.p.N;
  const bool by_element = pr.p.g.sw > 2;
  const long long long_k = by_element ? 768 : kConvLongK;
  int best = -1;
  long long best_area = 0;
  for (int c = 0; c < kNumConfigs; ++c) {
    const ConfigRow& r = kConfigs[c];
    if (r.sched != 3 || pr.p.K < r.bk || !find_launcher(pr, c)) continue;
    const long long area = (long long)r.bm * r.bn;
    const long long tiles = ((M + r.bm - 1) / r.bm) * ((N + r.bn - 1) / r.bn);
    const bool more = by_element && area == (M > 32 ? 64 * 32 : 32 * 32);
    // Of the 32x32 tile two workgroups share a compute unit: on a long K 512 of them beat the half-padded 64x64 tile and the
    // two-stage ones for 17 to 32 channels (28 images of 256x35x35, 32 channels, 5x5, stride 2, 378 tiles: 48 us, 64x64 55 us,
    // 32x64 of two stages 74 us; 64 of 256x28x28, 448 tiles: 44, 51 and 73 us).
    const bool pairs = M > 16 && M <= 32 && r.bm == 32 && r.bn == 32 && pr.p.K >= long_k;
    const long long round = pairs ? kComputeUnits * 2 : more ? kComputeUnits * 3 / 2 : kComputeUnits;
    if (tiles > round || tiles < kComputeUnits / 4) continue;
    if (area == 64 * 64 && pr.p.K >= long_k) {
      if (2 * M * N < tiles * area) continue;
    } else if (area == 128 * 64 && !by_element && pr.p.K >= 1408) {
      // (against 64x32 tiles of two stages, 380 random problems of 129 to 256 such tiles: 1.02-1.08 of the time at K =
      // 1152, even half padded 0.94 at 1440, 0.81 at 2304, 0.74 at 4608 and beyond)
      if (2 * M * N <= tiles * area || tiles < (pr.p.K >= long_k ? kComputeUnits / 2 : kComputeUnits * 3 / 4)) continue;
    } else if (area >= 64 * 64) {
      if (by_element ? 2 * M * N < tiles * area : 4 * M * N < 3 * tiles * area) continue;
      if (pr.p.K < long_k && (area == 64 * 64 || tiles < kComputeUnits * 3 / 4)) continue;
      if (area > 64 * 64 && tiles < kComputeUnits / 2) continue;
      // (half a round of 128x128 with a quarter of it padding loses to 64x32 of two stages where loads are by element: 37
      // images of 192x56x56, 192 channels, 3x3, stride 4: 111 and 76 us; 41 of 256x56x56, 320 channels: 146 and 159 us)
      if (by_element && area == 128 * 128 && 5 * M * N < 4 * tiles * area) continue;
    }
    // (of two tiles of one size the taller one: it gathers fewer columns)
    if (best < 0 || area < best_area || (area == best_area && r.bm > kConfigs[best].bm)) {
      best = c;
      best_area = area;
    }
  }
  return best;
}

// GEMMs in 16-bit types with few output tiles.  -1: more tiles than that, the choice below is made.
//
// Tiles whose wavefronts stream K (gemm_kernel_waves) keep a compute unit to themselves; one round of them costs a fixed
// 3 us and K times a rate that grows with the tile's extents, a second round as much again.  So the smallest one of
// which all workgroups are resident is taken (300x768x3072: 240 of 32x32 10.6 us, 60 of 64x64 15.5 us; 20.9 us on 16x16,
// which needs four rounds; 8x12288x4096, seven eighths of whose 64x64 tiles are padding: 23.4 us, 28.9 us on 16x32), on
// aligned rows a 16x16 one only if it leaves a quarter of the device free: a 16x32 one touches no more cache lines of a
// row-major B (117x512x2048: 256 of 16x16 6.8 us, 128 of 16x32 5.7 us; misaligned 276x213x3514: 10.9 and 11.9 us).  Each pays
// from the K on where its wavefronts have a step of their own, earlier where rows are only element aligned, which the other
// tiles fetch under predicates: measured against them on 320 random problems, 1.0 to 1.4 of their time below these limits, 0.4
// to 1.0 above.
// Below them the 32x32 tile of two stages, several to a compute unit, beats the larger ones as long as there are no more
// than three to a compute unit (1308x566x256, 738 tiles: 5.7 us, 64x64 8.7 us; 168x624x49: 3.9 us, 16x64 6.1 us), on aligned
// rows of more than 128 values the one of 256, of which a compute unit holds two (4 of 256x225x256: 4.6 us, 5.0 us).  From
// there to 384 tiles of 64x64 the tiles of half that size do, with loads one iteration ahead (320x4096x1024: 12.4 us on
// 32x64, 17.3 us on 128x128 K-splitting ones; 896x1246x72: 5.8 and 7.2 us on 64x64).
// Over 620 random problems of 1 to 4096 rows and columns this choice (with the one below) takes 1.01 times as long as the best
// configuration of each, the one before it 1.11 times; over 270 batched attention products 1.02 and 1.11.
int few_tiles_gemm_config(const Problem& pr) {
  constexpr long long kComputeUnits = 256;
  const long long M = pr.p.M, N = pr.p.N, K = pr.p.K;
  auto blocks = [&](long long bm, long long bn) { return sat_mul(((M + bm - 1) / bm) * ((N + bn - 1) / bn), pr.batch); };
  const long long of_64 = blocks(64, 64);
  if (of_64 >= 384) return -1;
  int best = -1;
  for (int c = 0; c < kNumConfigs; ++c) {
    const ConfigRow& r = kConfigs[c];
    if (r.sched != 3 || r.bm > 64 || r.bn > 64 || !find_launcher(pr, c)) continue;
    const int area = r.bm * r.bn;
    if (blocks(r.bm, r.bn) > (area == 16 * 16 && pr.elem_mode == 0 ? kComputeUnits * 3 / 4 : kComputeUnits)) continue;
    // (of two tiles of one size the flatter one: rows of B are M/N-contiguous more often than not)
    const int best_area = best < 0 ? 0 : kConfigs[best].bm * kConfigs[best].bn;
    if (best < 0 || area < best_area || (area == best_area && r.bn > kConfigs[best].bn)) best = c;
  }
  if (best >= 0) {
    const int area = kConfigs[best].bm * kConfigs[best].bn;
    if (K >= (area >= 64 * 64 ? 512 : area > 32 * 32 ? 448 : area == 32 * 32 || pr.elem_mode == 0 ? 257 : area > 16 * 16 ? 160 : 128))
      return best;
  }
  auto of_shape = [&](int bm, int bn, int bk, int sched) {
    for (int c = 0; c < kNumConfigs; ++c) {
      const ConfigRow& r = kConfigs[c];
      if (r.bm == bm && r.bn == bn && r.bk == bk && r.sched == sched && r.mfma == 16 && find_launcher(pr, c)) return c;
    }
    return -1;
  };
  if (blocks(32, 32) <= 3 * kComputeUnits) {
    const int deep = K > 128 && pr.elem_mode == 0 && blocks(32, 32) <= 2 * kComputeUnits ? of_shape(32, 32, 256, 0) : -1;
    return deep >= 0 ? deep : of_shape(32, 32, 64, 0);
  }
  const int halves = blocks(64, 32) <= blocks(32, 64) ? of_shape(64, 32, 64, 2) : of_shape(32, 64, 64, 2);
  return halves >= 0 ? halves : of_shape(32, 32, 64, 0);  // (a transposed A is built for the latter only)
}

// fp32 GEMMs with fewer than 384 tiles of 64x64, which are bound by latency: the tile with the shortest predicted time, a fixed
// time and a rate per value of K for the first 256 workgroups, and as much again in other shares for what there are beyond
// (whole rounds of the K-splitting ones, which keep a compute unit to themselves).  Fitted to 500 random products of 1 to 3000
// rows, columns and values of K, 5 % to 95 % of predictions over measurements 0.84 to 1.15.  Over 200 others this takes 1.008
// times as long as the best configuration of each; an order by tile size, as below, takes 1.11 times (854x27x203 9.1 -> 3.9 us, which
// took the 16x64 tile, 128x1136x1029 18.9 -> 10.7, which took half as many K-splitting ones; a transposed A of a long K, for
// which those are built as well, 16x40x1000 12.6 -> 4.9).
struct SmallF32Time {
  int bm, bn, bk, mfma, sched;
  struct {
    float fixed, per_k, more, more_per_k;  // us; of 1000 values of K
  } at[2];                                 // aligned rows, element-aligned ones
};
constexpr SmallF32Time kSmallF32Times[] = {{64, 64, 16, 32, 0, {{3.33f, 30.7f, 0.0f, 27.8f}, {3.73f, 30.9f, 1.79f, 21.5f}}},
                                           {64, 64, 16, 16, 0, {{3.47f, 26.3f, 0.0f, 28.1f}, {3.80f, 28.4f, 1.80f, 20.7f}}},
                                           {32, 32, 32, 16, 0, {{2.65f, 12.1f, 0.25f, 6.22f}, {2.80f, 13.6f, 0.53f, 6.33f}}},
                                           {32, 32, 32, 16, 2, {{2.74f, 9.73f, 0.20f, 6.96f}, {2.95f, 12.5f, 0.56f, 6.77f}}},
                                           {32, 32, 64, 16, 2, {{2.93f, 7.83f, 0.33f, 6.96f}, {3.29f, 10.1f, 0.86f, 6.24f}}},
                                           {32, 32, 128, 16, 3, {{3.31f, 6.35f, 1.64f, 6.06f}, {3.31f, 6.37f, 1.83f, 6.73f}}},
                                           {16, 16, 256, 16, 3, {{3.25f, 1.88f, 1.32f, 1.87f}, {3.23f, 1.64f, 1.35f, 2.39f}}},
                                           {16, 32, 256, 16, 3, {{3.19f, 3.65f, 1.25f, 3.77f}, {3.20f, 3.46f, 1.40f, 4.02f}}}};
int few_tiles_f32_config(const Problem& pr) {
  const long long M = pr.p.M, N = pr.p.N;
  if (sat_mul(((M + 63) / 64) * ((N + 63) / 64), pr.batch) >= 384) return -1;
  int best = -1;
  float best_us = 0.0f;
  for (int c = 0; c < kNumConfigs; ++c) {
    const ConfigRow& r = kConfigs[c];
    if (!r.is_f32 || !find_launcher(pr, c)) continue;
    for (const SmallF32Time& t : kSmallF32Times) {
      if (t.bm != r.bm || t.bn != r.bn || t.bk != r.bk || t.mfma != r.mfma || t.sched != r.sched) continue;
      const long long tiles = sat_mul(((M + r.bm - 1) / r.bm) * ((N + r.bn - 1) / r.bn), pr.batch);
      const float more = r.sched == 3 ? (float)((tiles + 255) / 256 - 1) : std::max(0.0f, (float)tiles / 256.0f - 1.0f);
      const auto& at = t.at[pr.elem_mode != 0];
      const float k = (float)pr.p.K / 1000.0f, us = at.fixed + at.per_k * k + more * (at.more + at.more_per_k * k);
      if (best < 0 || us < best_us) {
        best = c;
        best_us = us;
      }
    }
  }
  return best;
}

// Untuned choice: the largest tile that still gives (nearly) every compute unit a workgroup, else the largest
// that gives a quarter of them one, else the tile with the most workgroups.  Outputs large enough to be bound by
// throughput rather than by one workgroup's latency chain (at least 384 tiles of 64x64) ask for about two
// workgroups per compute unit instead, so that one workgroup's loads and output write overlap another's
// arithmetic -- except from the ring schedule on four or more stages of K, which overlaps them inside the
// workgroup and needs just over half a round of workgroups.  Between tiles of one size the ring schedule, the
// 16x16 matrix-core shape and (small tiles) the loads-ahead order are preferred (they measure faster wherever
// both apply); the tiles that split K over wave groups take part only when K spans at least one of their K tiles
// and the output is small (GEMMs: few_tiles_gemm_config and few_tiles_f32_config alone take them).  With slices > 1 only tiles
// that have a K-parallel form take part.
int default_config(const Problem& pr, int slices = 1) {
  const long long M = pr.p.M, N = pr.p.N;
  const bool conv16 = pr.op == 1 && pr.dtype != HIDET_F32 && slices <= 1;
  if (conv16 && pr.p.K >= 512) {
    const int c = one_round_config(pr);
    if (c >= 0) return c;
  }
  const bool gemm16 = pr.op == 0 && pr.dtype != HIDET_F32 && slices <= 1;
  if (pr.op == 0 && slices <= 1) {
    const int c = gemm16 ? few_tiles_gemm_config(pr) : few_tiles_f32_config(pr);
    if (c >= 0) return c;
  }
  // The gather of a convolution is paid per column of the tile, and fewer than 64 output channels fill one tile row
  // anyway: there the 64x64 tile, more of which are resident together, beats the wider and the padded ones, with 32x32
  // matrix-core tiles once it is bound by throughput (64 images of 64x56x56, 3x3: 66 us on 64x128, 54 us on 64x64 of
  // 16x16, 50 us of 32x32).
  // (Not measured for repacked weights, whose gather is cheaper.)
  const bool conv_few_rows = conv16 && M <= 64 && !pr.packed;
  // (measured: equal to the two-stage tiles of their size at K = 1024, ahead beyond; the gather of the convolution
  // moves that point to about 512)
  const bool long_k = pr.p.K >= (pr.op == 1 ? 512 : 1024);
  // (loads one iteration ahead: measured faster on small tiles only, and of a GEMM on aligned rows only -- predicated
  // loads wait where they are issued: 184 of 103x128x103 10.5 us, 6.8 us without)
  const bool ahead_pays = pr.op == 1 || pr.elem_mode == 0;
  auto rank = [long_k, ahead_pays](const ConfigRow& r) {
    const int ahead = (r.sched == 2 && r.bm * r.bn <= 64 * 64 && ahead_pays) ? 1 : 0;
    const int ksplit = (r.sched == 3 && long_k) ? 2 : 0;  // where they take part at all, they win on a long K
    return (long long)r.bm * r.bn * 8 + (r.sched == 1 ? 4 : 0) + (r.mfma == 16 ? 2 : 0) + ahead + ksplit;
  };
  const bool throughput = sat_mul(((M + 63) / 64) * ((N + 63) / 64), pr.batch) >= 384;
  // (tile extents are powers of two, so that this choice, made on every call that names no configuration, shifts
  // where it would divide)
  int best = -1, fewer = -1, most = -1, passed_over = -1;
  long long most_blocks = -1, best_key = -(1LL << 62), fewer_key = -(1LL << 62);
  for (int c = 0; c < kNumConfigs; ++c) {
    if (!find_launcher(pr, c)) continue;
    if (slices > 1 && !find_partial_launcher(pr, c)) continue;
    const ConfigRow& r = kConfigs[c];
    // the wave groups along K need at least one whole K tile to share, and are meant for latency-bound problems
    if (r.sched == 3 && (pr.p.K < r.bk || throughput || gemm16)) continue;
    if (conv_few_rows && (r.bm > 64 || r.bn > 64)) {
      passed_over = c;
      continue;
    }
    const long long tiles = ((M + r.bm - 1) >> __builtin_ctz(r.bm)) * ((N + r.bn - 1) >> __builtin_ctz(r.bn));
    const long long blocks = sat_mul(tiles, pr.batch * (slices > 1 ? slices : 1));
    // (a convolution: what one round of them can do has been decided above; the small ones, of which a compute unit holds
    // two, still win a little beyond it for few channels on a long K: 43 images of 512x28x28, 24 channels, 3x3, stride 2:
    // 41 us on 301 of 32x32, 50 us on two-stage tiles)
    const long long resident = conv16 && M <= 32 && r.bm * r.bn <= 32 * 32 && pr.p.K >= kConvLongK ? 640 : 256;
    if (conv16 && r.sched == 3 && (blocks > resident || (pr.p.K >= 512 && (long long)r.bm * r.bn >= 64 * 64))) {
      passed_over = c;
      continue;
    }
    // the ring schedule runs GEMMs only: by direct-to-LDS loads (at any element alignment), with its stages
    // staged through registers when an input prologue has to touch the values
    const bool ring_any = r.sched == 1 && pr.op == 0 && pr.p.out_map == 0;
    const bool ring = ring_any && pr.p.relu_a == 0 && pr.p.relu_b == 0;
    // A ring tile keeps one workgroup per compute unit busy on its own (from four stages of K on).  With 129..191
    // of them the tile of half the size would need a second, mostly empty round of workgroups, so the larger one is
    // still the better choice; from 128 down the smaller tile fits into one round and wins.
    // (a quarter of it padding in every entry of a batch, no large tile is: 88 of 400x64x400 15.2 us on 256x128 tiles, 10.2
    // us on 64x64; 65 of 398x398x128 29.9 us on 256x256, 17.2 us; 84 of 448x448x128 28.1 and 16.7 us)
    const long long area = (long long)r.bm * r.bn;
    // (half of one is enough on a long K, and on element-aligned rows for 128x128 tiles, against which smaller ones load under
    // predicates: 78 of 96x729x512 19.3 us on 128x256, 30.9 us on 32x64; 111 of 88x511x42 8.4 us on 128x128, 11.6 us on 32x64)
    const bool half_pays = pr.p.K >= 256 || (area == 128 * 128 && pr.elem_mode != 0);
    const long long full = area >= 256 * 256 && pr.p.K <= 128 ? 7 : half_pays ? 4 : 6;  // eighths of a tile that have to be output
    if (gemm16 && pr.batch > 1 && area >= 128 * 128 && 8 * M * N <= full * tiles * area) {
      passed_over = c;
      continue;
    }
    // (nor does a batch take the 16x64 tile, two wavefronts that need as long as the four of a 32x64 one: 96 of 48x196x1024
    // 46.3 and 22.8 us, 148 of 48x169x64 10.7 and 5.1 us, 94 of 10x358x36 8.1 and 4.7 us; but for aligned rows and no more
    // than 16 of them, 40 of 16x1600x256: 6.1 and 6.9 us)
    if (gemm16 && pr.batch > 1 && r.bm == 16 && r.bn == 64 && (M > 16 || pr.elem_mode != 0)) {
      passed_over = c;
      continue;
    }
    // (nor, into rows that are only element aligned, a 128x64 or 64x128 one: 128 of 327x327x32 18.6 and 18.8 us, 17.5 us on
    // 64x64; 64 of 255x255x128 8.0, 8.1 and 7.1 us; 190 of 191x191x128 13.4, 13.9 and 10.3 us)
    if (gemm16 && pr.batch > 1 && pr.p.vec_store < 2 && pr.p.out_map == 0 && area == 128 * 64) {
      passed_over = c;
      continue;
    }
    const bool self_overlapping = ring_any && pr.p.K >= 4 * r.bk;
    const long long enough = !throughput ? 192 : self_overlapping ? 129 : gemm16 ? 384 : 400;
    // Tiles of 64x64 and more are no first choice of a convolution outside the rule above that is bound by latency (fewer
    // than 384 of them: 7 images of 64x56x56, 5x5: 343 tiles of 64x64 26.5 us, 64x32 21.8 us; 9 images of 128x28x28, 3x3:
    // 18.3 us and 14.8 us).  From 64x32 down one round is enough (18 images of 128x28x28 repacked, stride 2: 64x32 13.5
    // us, 32x32 15.4 us).
    const bool large = conv16 && !throughput && area >= 64 * 64;

    // useful outputs per workgroup, discounted by the share of the tile that is padding, decide; then the smaller
    // tile, then the schedule preferences
    const long long useful = (M * N) / tiles;
    long long weight = (useful * useful) >> __builtin_ctzll(area);
    // (of a batch, whose entries are all cut alike, by the sixth power of the share that is output: 96 of 320x320x32 10.6 us
    // on 128x64 tiles five sixths full, 8.1 us on 64x64; 43 of 448x448x64 10.0 and 8.4 us)
    if (gemm16 && pr.batch > 1) {
      const long long fill = (useful << 10) >> __builtin_ctzll(area), square = (fill * fill) >> 10;
      weight = (((weight * square) >> 10) * square) >> 10;
    }
    // (the 64x64 tile alone: the 32x32 one of that matrix-core shape is a single wavefront with a deep K tile; 8 images of
    // 16x112x112, 24 channels, 3x3, stride 2: 10.1 us on it, 7.5 us on the 32x32 tile of 16x16)
    // Not on a long K while the tiles of three stages, three to a compute unit, are all resident at once: the third stage
    // hides the gather better, most of all a strided one (40 images of 192x56x56, 64 channels, 5x5, stride 2, 560 tiles: 102
    // us on 32x32 of two stages, 96 us on 16x16 of three; 16 tiles more than 768 are a second round, 1.15 times slower
    // than two stages).  With stride 1 this ends at two to a compute unit (384-512 tiles: 0.99 of the time, 513-768: 1.02).
    const bool all_resident = long_k && tiles <= (pr.p.g.sw > 1 ? 768 : 512);
    const long long preference =
        (conv_few_rows && throughput && !all_resident && r.mfma == 32 && area == 64 * 64) ? 8 : rank(r) & 63;
    long long key = weight * (1LL << 23) - area * 64 + preference;
    // a K of at most two stages runs the two-slot ring: two workgroups of a 256x128 tile share a compute unit and
    // outrun one of a 256x256 tile
    if (ring && pr.p.K <= 2 * r.bk && area == 256 * 128) key += weight * (3LL << 22);
    // of the two rectangular ring tiles the one of 128 rows, if it needs no round more, where B is row-major: each stage reads half
    // as many pieces of 64 bytes of A's rows for it, and longer ones of B's (140 random products of 1200 to 4000: 0.93 of the
    // time of 256x128 on aligned rows, 0.89 with an odd K, 0.85 with odd extents, 1.02 where both operands are read along K)
    if (ring && gemm16 && pr.batch == 1 && !pr.transB && pr.p.K > 2 * r.bk && r.bm == 128 && r.bn == 256) {
      const long long upright = ((M + 255) >> 8) * ((N + 127) >> 7);
      if ((tiles + 255) >> 8 <= (upright + 255) >> 8) key += weight * (1LL << 21);
    }
    // (the gather is paid once per row of tiles, so a flat tile is the last resort of a convolution of more rows: 7 images
    // of 192x28x28, 72 channels, 3x3: 26.5 us on three rows of 32x64 tiles, 20 us on two of 64x32)
    const bool flat = conv16 && M > 64 && r.bm < 64 && r.bn >= 64;
    if (blocks >= enough && key > best_key && !flat && !large) {
      best = c;
      best_key = key;
    }
    // second choice when no tile gives that many workgroups: the same order among the tiles that still give 64
    if (blocks >= 64 && key > fewer_key && !flat) {
      fewer = c;
      fewer_key = key;
    }
    // last resort (not even 64 workgroups): the most workgroups; between equals the smaller tile, then the deeper K
    // tile that K still fills (one workgroup's latency chain is all there is to shorten), then the preferences
    auto beats = [&](const ConfigRow& a, const ConfigRow& b) {
      if (a.bm * a.bn != b.bm * b.bn) return a.bm * a.bn < b.bm * b.bn;
      const int ka = a.bk <= pr.p.K ? a.bk : 0, kb = b.bk <= pr.p.K ? b.bk : 0;
      if (ka != kb) return ka > kb;
      return rank(a) > rank(b);
    };
    if (blocks > most_blocks || (blocks == most_blocks && beats(r, kConfigs[most]))) {
      most_blocks = blocks;
      most = c;
    }
  }
  return best >= 0 ? best : fewer >= 0 ? fewer : most >= 0 ? most : passed_over;
}

// ---- static scratch of the allocation-free K-parallel entry point --------------------------------------
// One array per GPU, part of the code object, held until the process ends.  In host code the array's name is only
// a handle: the device address is asked for once per device (with that device current) and kept.
constexpr long long kScratchBytes = 32LL << 20;
constexpr int kMaxDevices = 64;
__device__ __attribute__((aligned(256))) unsigned char g_scratch[kScratchBytes];
void* g_scratch_ptr[kMaxDevices] = {};

// ---- tuned-config cache ---------------------------------------------------------------------------
std::mutex g_mutex;

hidet_status_t scratch_of_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return HIDET_ERR_LAUNCH;
  std::lock_guard<std::mutex> lock(g_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_scratch)) != hipSuccess || !ptr) return HIDET_ERR_LAUNCH;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return HIDET_OK;
}
struct Tuned {
  int config;  // of the form; of the fastest gather with the patch forms, which have none
  int slices;
  int form = HIDET_CONV_GATHER;  // convolutions only
};
std::map<std::string, Tuned> g_cache;
std::vector<float> g_last_times;

std::string problem_key(const Problem& pr, bool with_workspace = false) {
  char buf[256];
  const GemmParams& p = pr.p;
  const int epi_kind = p.bias_axis | (p.residual ? 4 : 0) | (p.relu ? 8 : 0) | (p.alpha != 1.0f ? 16 : 0) |
                       (p.out_map ? 32 : 0) | (pr.wide_out ? 64 : 0) | ((p.relu_a || p.relu_b) ? 128 : 0);
  if (pr.op == 0)
    std::snprintf(buf, sizeof(buf), "gemm:t%d:%d%d:b%lld:%dx%dx%d:e%d:m%d", pr.dtype, pr.transA, pr.transB, pr.batch, p.M,
                  p.N, p.K, epi_kind, pr.elem_mode);
  else
    std::snprintf(buf, sizeof(buf), "conv:t%d:n%lld:c%d:%dx%d:o%lld:k%dx%d:s%dx%d:p%dx%d:e%d:m%d%s", pr.dtype, pr.Nb, p.g.IC,
                  p.g.H, p.g.W, pr.OC, p.g.KH, p.g.KW, p.g.sh, p.g.sw, p.g.ph, p.g.pw, epi_kind, pr.elem_mode,
                  pr.packed ? ":pk" : "");
  return std::string(buf) + (with_workspace ? ":ws" : "");
}

struct SplitK {  // how the caller wants K parallelised
  int slices = 1;            // requested number of K slices (<= 1: none); < 0 with a workspace: take the tuned value
  void* workspace = nullptr;
  long long workspace_bytes = 0;
  bool fixed = false;  // the workspace is the library's static scratch array: too small is HIDET_ERR_SCRATCH
};

// (g_mutex held.)  A process that has tuned nothing does not print keys: that took over a microsecond of each call.
std::map<std::string, Tuned>::const_iterator find_tuned(const Problem& pr, const SplitK& sk) {
  return g_cache.empty() ? g_cache.end() : g_cache.find(problem_key(pr, sk.workspace != nullptr));
}

template <int MAPPER>
hipError_t reduce_dispatch(int dtype, const GemmParams& p, int batch, hipStream_t stream) {
  switch (dtype) {
    case HIDET_F32: return launch_reduce<float, MAPPER>(p, batch, stream);
    case HIDET_F16: return launch_reduce<f16, MAPPER>(p, batch, stream);
    default: return launch_reduce<bf16, MAPPER>(p, batch, stream);
  }
}

thread_local long long g_kernel_launches = 0;  // GEMM / convolution kernels this thread has launched so far

// The part of a GEMM (rows or columns, a multiple of 256) that the 256x256 ring tile should take when the rest is
// better served by a smaller tile; none if both extents are 0.  With T tiles of 256x256, T / 256 whole rounds keep
// every compute unit busy; a thin last round leaves most of the device idle for 0.6 of a tile's time (measured: it
// runs at a higher clock than a full round).  At most 64 left-over tiles make at most 256 tiles of 128x128, one
// round that takes 0.3 to 0.45 of that time; more of them would need the 128x256 tile (0.6: no gain) or a second
// round.  Measured, 4352^3: 196 -> 154 us; 7168^3: 643 -> 602 us.  The cut is made along M or along N, whichever
// leaves fewer tiles over.
struct RoundCut {
  long long rows = 0, cols = 0;  // at most one is non-zero: extent of the head along M or along N
};
RoundCut cut_for_whole_rounds(const Problem& pr, int config, int slices) {
  RoundCut cut;
  const ConfigRow& r = kConfigs[config];
  const GemmParams& p = pr.p;
  if (pr.op != 0 || pr.batch != 1 || slices > 1 || p.out_map != 0) return cut;
  if (r.sched != 1 || r.bm != 256 || r.bn != 256) return cut;
  const long long tm = (p.M + 255) / 256, tn = (p.N + 255) / 256, tiles = tm * tn;
  const long long whole = tiles / 256;
  if (whole < 1 || tiles % 256 == 0) return cut;
  // tile rows (columns) that fit into the whole rounds, and the 256x256 tiles left over
  const long long head_rows = whole * 256 / tn, head_cols = whole * 256 / tm;
  const long long rest_rows = head_rows >= 1 && head_rows < tm ? (tm - head_rows) * tn : -1;
  const long long rest_cols = head_cols >= 1 && head_cols < tn ? (tn - head_cols) * tm : -1;
  // (at most 64: one round of 128x128 tiles)
  const bool rows_ok = rest_rows >= 0 && rest_rows <= 64, cols_ok = rest_cols >= 0 && rest_cols <= 64;
  if (rows_ok && (!cols_ok || rest_rows <= rest_cols))
    cut.rows = head_rows * 256;
  else if (cols_ok)
    cut.cols = head_cols * 256;
  return cut;
}

hidet_status_t launch(const Problem& pr_in, int config, const SplitK& sk, hipStream_t stream) {
  Problem pr = pr_in;
  GemmParams& p = pr.p;
  if (pr.batch == 0 || p.M == 0 || p.N == 0) return HIDET_OK;
  int slices = sk.slices;
  if (config < 0) {
    {
      std::lock_guard<std::mutex> lock(g_mutex);
      auto it = find_tuned(pr, sk);
      if (it != g_cache.end()) {
        config = it->second.config;
        if (slices < 0) slices = it->second.slices;
      }
    }
    if (slices < 0) slices = 1;
    // (a remembered configuration that has no K-parallel form cannot serve an explicit slice count)
    if (config < 0 || !find_launcher(pr, config) || (slices > 1 && !find_partial_launcher(pr, config)))
      config = default_config(pr, slices);
    // A GEMM for which the caller named no configuration (size-based or remembered choice), on the 256x256 ring
    // tile, whose tiles fill whole rounds of the 256 compute units plus a thin last round (at most a quarter full):
    // the tile rows (or columns) that make up the whole rounds run as they are, the remaining ones run as a problem
    // of their own, for which the size-based choice takes a smaller tile that fills the device.  Two launches on
    // the same stream, no partial sums: every output element is still computed by one workgroup over all of K.
    const RoundCut cut = config >= 0 ? cut_for_whole_rounds(pr, config, slices) : RoundCut();
    if (cut.rows > 0 || cut.cols > 0) {
      Problem head = pr, tail = pr;
      const long long es_in = elem_size(pr.dtype), es_out = pr.wide_out ? 4 : es_in;
      if (cut.rows > 0) {
        const long long rows = cut.rows;
        head.p.M = (int)rows;
        tail.p.M = p.M - (int)rows;
        tail.p.A = static_cast<const char*>(p.A) + (pr.transA ? rows : rows * p.lda) * es_in;
        tail.p.C = static_cast<char*>(p.C) + rows * p.ldc * es_out;
        if (p.residual) tail.p.residual = static_cast<const char*>(p.residual) + rows * p.ldr * es_out;
        if (p.bias && p.bias_axis == 2) tail.p.bias = static_cast<const char*>(p.bias) + rows * es_out;
      } else {
        const long long cols = cut.cols;
        head.p.N = (int)cols;
        tail.p.N = p.N - (int)cols;
        tail.p.B = static_cast<const char*>(p.B) + (pr.transB ? cols * p.ldb : cols) * es_in;
        tail.p.C = static_cast<char*>(p.C) + cols * es_out;
        if (p.residual) tail.p.residual = static_cast<const char*>(p.residual) + cols * es_out;
        if (p.bias && p.bias_axis == 1) tail.p.bias = static_cast<const char*>(p.bias) + cols * es_out;
      }
      // the rest's configuration is settled before anything is launched: a call that fails has written nothing
      const int tail_config = default_config(tail, 1);
      if (tail_config >= 0 && find_launcher(tail, tail_config) && find_launcher(head, config)) {
        const hidet_status_t st = launch(head, config, sk, stream);
        return st != HIDET_OK ? st : launch(tail, tail_config, sk, stream);
      }
    }
  }
  if (slices < 0) slices = 1;
  LaunchFn fn = find_launcher(pr, config);
  if (!fn) return HIDET_ERR_NO_CONFIG;
  const ConfigRow& r = kConfigs[config];
  const int tiles_m = (p.M + r.bm - 1) / r.bm, tiles_n = (p.N + r.bn - 1) / r.bn;
  // grouped traversal: each run of 32 consecutive workgroups (one die's share of a 256-tile wave)
  // should cover a near-square patch of tiles
  set_block_mapping(p, tiles_m, tiles_n, tiles_m >= 4 ? 4 : tiles_m);
  p.k_slices = 1;
  p.k_slice_len = p.K;
  long long len = p.K, actual = 1;
  if (slices > 1 && p.K > 0) {
    len = (p.K + slices - 1) / slices;
    len = (len + r.bk - 1) / r.bk * r.bk;  // whole K tiles per slice keeps every slice 16-byte aligned
    actual = (p.K + len - 1) / len;
  }
  if (actual <= 1) {
    const long long total = sat_mul((long long)p.tiles_m * p.tiles_n, pr.batch);
    if (total > kIntMax) return HIDET_ERR_UNSUPPORTED;
    p.total_blocks = (int)total;
    if (fn(p, stream) != hipSuccess) return HIDET_ERR_LAUNCH;
    ++g_kernel_launches;
    return HIDET_OK;
  }
  // ---- parallel reduction on K: partial sums into the workspace, then reduce + epilogue
  LaunchFn pfn = find_partial_launcher(pr, config);
  if (!pfn) return HIDET_ERR_NO_CONFIG;
  if (pr.batch > 65535) return HIDET_ERR_UNSUPPORTED;
  const long long total = sat_mul((long long)p.tiles_m * p.tiles_n, pr.batch * actual);
  if (total > kIntMax) return HIDET_ERR_UNSUPPORTED;
  const long long need = sat_mul(sat_mul(4LL * pr.batch * actual, p.M), p.N);
  if (sk.fixed && sk.workspace_bytes < need) return HIDET_ERR_SCRATCH;
  if (!sk.workspace || sk.workspace_bytes < need) return HIDET_ERR_INVALID_ARG;
  if (!aligned(sk.workspace, 16)) return HIDET_ERR_ALIGNMENT;
  GemmParams q = p;
  q.C = sk.workspace;
  q.ldc = p.N;
  q.strideC = (long long)p.M * p.N;
  q.alpha = 1.0f;
  q.bias = nullptr;
  q.bias_axis = 0;
  q.residual = nullptr;
  q.relu = 0;
  q.out_map = 0;
  q.vec_store = (p.N % 4 == 0) ? 2 : 1;
  q.k_slices = (int)actual;
  q.k_slice_len = (int)len;
  q.total_blocks = (int)total;
  q.out_inner = 1;
  q.out_outer = 0;
  if (pfn(q, stream) != hipSuccess) return HIDET_ERR_LAUNCH;
  ++g_kernel_launches;
  GemmParams rp = p;
  rp.A = sk.workspace;
  rp.k_slices = (int)actual;
  const int out_type = pr.wide_out ? (int)HIDET_F32 : pr.dtype;
  const hipError_t e = pr.op == 1 ? reduce_dispatch<MAP_NCHW>(out_type, rp, (int)pr.batch, stream)
                                  : reduce_dispatch<MAP_PLAIN>(out_type, rp, (int)pr.batch, stream);
  if (e == hipSuccess) ++g_kernel_launches;
  return e == hipSuccess ? HIDET_OK : HIDET_ERR_LAUNCH;
}

const int kSliceChoices[] = {1, 2, 3, 4, 6, 8, 12, 16};

// Times `iters` launches in a row on a stream.
class Stopwatch {
 public:
  Stopwatch(hipStream_t stream, int iters) : stream_(stream), iters_(iters > 0 ? iters : 10) {
    if (hipEventCreate(&e0_) != hipSuccess) e0_ = nullptr;
    if (hipEventCreate(&e1_) != hipSuccess) e1_ = nullptr;
  }
  ~Stopwatch() {
    if (e0_) (void)hipEventDestroy(e0_);
    if (e1_) (void)hipEventDestroy(e1_);
  }
  Stopwatch(const Stopwatch&) = delete;
  Stopwatch& operator=(const Stopwatch&) = delete;
  bool ready() const { return e0_ && e1_; }
  // Mean microseconds of `run` after a first one, which also loads the code object; -1 where it refuses.  False: the stream failed.
  template <class F>
  bool time(F run, float* us) {
    *us = -1.0f;
    if (run() != HIDET_OK) return true;
    (void)hipEventRecord(e0_, stream_);
    for (int i = 0; i < iters_; ++i) run();
    (void)hipEventRecord(e1_, stream_);
    if (hipEventSynchronize(e1_) != hipSuccess) return false;
    float ms = 0.0f;
    (void)hipEventElapsedTime(&ms, e0_, e1_);
    *us = ms * 1000.0f / (float)iters_;
    return true;
  }

 private:
  hipStream_t stream_;
  int iters_;
  hipEvent_t e0_ = nullptr, e1_ = nullptr;
};

// Enumerates the schedule space (x the K-slice choices when a workspace is given) on the caller's fused problem.
hidet_status_t tune(const Problem& pr, const SplitK& sk, hipStream_t stream, int iters, int32_t* best_config,
                    int32_t* best_slices, float* best_us) {
  std::vector<float> times(kNumConfigs, -1.0f);
  int best = -1, best_sl = 1;
  float best_t = 0.0f;
  if (!(pr.batch == 0 || pr.p.M == 0 || pr.p.N == 0)) {
    Stopwatch watch(stream, iters);
    if (!watch.ready()) return HIDET_ERR_LAUNCH;
    for (int c = 0; c < kNumConfigs; ++c) {
      if (!find_launcher(pr, c)) continue;
      for (int sl : kSliceChoices) {
        if (sl > 1 && !sk.workspace) break;
        SplitK one = sk;
        one.slices = sl;
        float us = 0.0f;
        if (!watch.time([&] { return launch(pr, c, one, stream); }, &us)) return HIDET_ERR_LAUNCH;
        if (us < 0.0f) continue;
        if (times[c] < 0.0f || us < times[c]) times[c] = us;
        if (best < 0 || us < best_t) {
          best = c;
          best_sl = sl;
          best_t = us;
        }
      }
    }
    if (best < 0) return HIDET_ERR_NO_CONFIG;
    // leave the winner's output in the buffer
    SplitK win = sk;
    win.slices = best_sl;
    launch(pr, best, win, stream);
    (void)hipStreamSynchronize(stream);
  }
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    if (best >= 0) g_cache[problem_key(pr, sk.workspace != nullptr)] = Tuned{best, best_sl, 0};
    g_last_times = times;
  }
  if (best_config) *best_config = best;
  if (best_slices) *best_slices = best_sl;
  if (best_us) *best_us = best_t;
  return HIDET_OK;
}

// No C++ exception crosses the C boundary: the cache and the tuner allocate host memory (strings, a map, a
// vector), and a failed allocation is reported as a failed launch.
template <class F>
hidet_status_t guarded(F f) noexcept {
  try {
    return f();
  } catch (...) {
    return HIDET_ERR_LAUNCH;
  }
}

// ---- convolution calls ------------------------------------------------------------------------------------------
// A 1x1 convolution with unit stride and no padding needs no gather: image b of x is an IC x (H*W) row-major
// matrix as it stands, so y[b] = w . x[b] is a batched GEMM with the weights shared across the batch (and the
// aligned direct-to-LDS loads of the ring schedule apply).  Such a call carries both descriptions of the problem.
struct ConvCall {
  Problem conv, gemm;
  bool pointwise = false;
};

// The configuration of a 1x1 convolution as one product whose columns run through all images; -1: this form cannot run it.
// (A K slice or an input prologue needs another kernel; direct loads need aligned weights, and rows of a chunk at least, so
// that one leaves the tensor in the last stage alone; their offsets from the tile's first image are 32 bits wide.)
int images_form(const Problem& conv, bool pointwise, const SplitK& sk) {
  const ConvGeom& g = conv.p.g;
  if (!pointwise || conv.dtype == HIDET_F32 || conv.elem_mode != 0 || conv.p.relu_b != 0 || sk.slices > 1) return -1;
  if (conv.p.K == 0 || conv.p.N == 0 || conv.p.M == 0 || g.HW < 8) return -1;
  if ((128 / g.HW + 2) * (long long)g.IC * g.HW > (1LL << 30)) return -1;
  for (int c = 0; c < kNumConfigs; ++c)
    if (registry().fn[c][conv.dtype][kPointwiseVariant]) return c;
  return -1;
}
// Microseconds of a batched GEMM on the tile that would be taken, and of the product over all images: predictions for the choice
// between the two alone.  A fixed time, one for each wave of resident workgroups where that shows, and for each round of 256
// workgroups (whole ones of ring tiles) the time of a workgroup's output, of its residual and of 32 values of K.  Fitted to
// 3300 random convolutions of 16 to 2048 channels: 5 % to 95 % of predictions over measurements 0.8 to 1.15, of the product
// 0.84 to 1.18.
struct BatchedTime {
  int bm, bn, ring, resident;  // ring: 1 with a K of at most two stages (two workgroups to a compute unit), 2 beyond
  double fixed, wave, out, residual, per_k;  // us
};
constexpr BatchedTime kAlignedTimes[] = {
    {32, 32, 0, 1, 4, 0, 0, 0.1, 0.085},         {16, 64, 0, 1, 4, 0, 0.5, 0.2, 0.11},        {64, 32, 0, 1, 4, 0, 0.33, 0.1, 0.092},
    {32, 64, 0, 1, 4, 0, 0.42, 0.15, 0.095},     {64, 64, 0, 5, 3.1, 2.1, 0.18, 0.33, 0.154}, {128, 64, 0, 3, 3.9, 2.6, 0.67, 0.66, 0.19},
    {64, 128, 0, 3, 3.2, 3.6, 0.4, 0.94, 0.22},  {128, 128, 1, 1, 4, 0, 3, 0.8, 0.32},        {256, 128, 1, 1, 4, 0, 4.7, 4.1, 0.64},
    {128, 256, 1, 1, 4, 0, 5.6, 3.1, 0.6},       {256, 256, 1, 1, 4, 0, 14, 11.2, 0.64},      {128, 128, 2, 1, 2, 0, 4.4, 1.7, 0.279},
    {256, 128, 2, 1, 1.6, 0, 7.9, 4.9, 0.523},   {128, 256, 2, 1, 1.3, 0, 8.6, 4.9, 0.478},   {256, 256, 2, 1, 4, 0, 14, 11.2, 0.64}};
constexpr BatchedTime kElementTimes[] = {
    {32, 32, 0, 1, 4, 0, 0.12, 0.1, 0.107},      {16, 64, 0, 1, 4, 0, 1.2, 0.3, 0.16},        {64, 32, 0, 1, 4, 0, 0.35, 0.2, 0.135},
    {32, 64, 0, 1, 4, 0, 0.52, 0.17, 0.155},     {64, 64, 0, 1, 4, 0, 0.95, 0.43, 0.21},      {128, 64, 0, 1, 4, 0, 3.3, 0.9, 0.25},
    {64, 128, 0, 1, 4, 0, 2.7, 1.4, 0.28},       {128, 128, 1, 1, 4, 0, 2.8, 1.5, 0.39},      {256, 128, 1, 1, 4, 0, 5.2, 4.3, 0.69},
    {128, 256, 1, 1, 4, 0, 5.7, 5.4, 0.7},       {256, 256, 1, 1, 4, 0, 15, 12.6, 0.68},      {128, 128, 2, 1, 1.9, 0, 6.1, 2, 0.288},
    {256, 128, 2, 1, 2.9, 0, 8.5, 5.7, 0.544},   {128, 256, 2, 1, 2.2, 0, 9.3, 6.2, 0.492},   {256, 256, 2, 1, 4, 0, 15, 12.6, 0.68}};
double batched_us(const Problem& gemm) {
  const int c = default_config(gemm);
  if (c < 0 || kConfigs[c].sched == 3) return 0.0;  // (K-splitting tiles: few of them, not compared)
  const ConfigRow& r = kConfigs[c];
  const int ring = r.sched != 1 ? 0 : gemm.p.K <= 2 * r.bk ? 1 : 2;
  const long long tiles = sat_mul(gemm.batch, sat_mul((gemm.p.M + r.bm - 1) / r.bm, (gemm.p.N + r.bn - 1) / r.bn));
  const BatchedTime* const times = gemm.elem_mode != 0 ? kElementTimes : kAlignedTimes;
  static_assert(sizeof(kElementTimes) == sizeof(kAlignedTimes), "the same tiles");
  for (size_t i = 0; i < sizeof(kAlignedTimes) / sizeof(kAlignedTimes[0]); ++i) {
    const BatchedTime& t = times[i];
    if (t.bm != r.bm || t.bn != r.bn || t.ring != ring) continue;
    const double rounds = ring ? (double)((tiles + 255) >> 8) : std::max(1.0, (double)tiles / 256.0);
    const long long resident = 256LL * t.resident;
    return t.fixed + t.wave * (double)((tiles + resident - 1) / resident) +
           rounds * (t.out + (gemm.p.residual ? t.residual : 0.0) + t.per_k * gemm.p.K / 32.0);
  }
  return 0.0;
}
double images_us(const Problem& conv, long long tiles) {  // (two workgroups to a compute unit; one alone takes 1.5 times its half)
  const double rounds = std::max(1.5, (double)((tiles + 255) >> 8));
  return 2.4 + rounds * (2.5 + (conv.p.residual ? 0.3 : 0.0) + 0.284 * conv.p.K / 32.0);
}

// A 1x1 convolution as one product whose columns run through all images (pixels of an image rounded up to whole chunks of
// eight), on the 128x128 ring tile with stages of 32, two workgroups to a compute unit: the configuration, or -1 where the
// batched GEMM is taken.  Against it there is no padding of every image to whole tiles, rows of 49 or 169 pixels come in by
// direct loads, the weights are read once per 128 columns and the residual is fetched at once (64 images of 512x7x7, 2048
// channels, with residual: 37.7 -> 18.4 us; 64 of 128x28x28, 512 channels, with residual: 66 -> 34 us; 57 of 192x21x21, 336
// channels: 25 -> 17 us).
// It wants more than half a round of tiles, a whole one where the batched GEMM has aligned rows (110 random problems, its time
// over the GEMM's: 0.42 to 1.04 from 120 tiles on rows that are not, but 1.2 at 69 to 80; on aligned ones 0.43 to 0.89 beyond
// 256 tiles, 1.15 at 208), and twice two rounds where half of a tile or more is padding (64 channels: 0.8 at 518 tiles, 1.1 at
// 417; 32 channels 1.35 at 356, 0.67 at 627).
// The counts know neither the batched GEMM's tile nor its rounds: where the predictions say that it is faster by a twelfth (of
// K = 64 they are no better than that) it is taken.  Of 3300 random convolutions 295 were more than 4 % slower than through it
// by the counts alone (64 images of 1024x14x14, 256 channels: 16.6 and 19.0 us; 125 of 2048x14x14, 512 channels: 64 and 79 us;
// 65 of 192x32x32, 32 channels: 7.8 and 13.1 us; 26 of 64x56x56, 64 channels: 9.4 and 12.6 us), 139 are now, by a quarter at
// most (95 of 64x11x11, 160 channels: 6.0 and 7.5 us); of the others 18 lost as much (32 of 64x56x56, 64 channels: 12.7 and
// 14.2 us).
int images_config(const ConvCall& cc, const SplitK& sk) {
  const Problem& conv = cc.conv;
  const int c = images_form(conv, cc.pointwise, sk);
  if (c < 0) return -1;
  const ConvGeom& g = conv.p.g;
  const long long tiles = (((long long)conv.p.M + 127) >> 7) * ((conv.Nb * ((g.HW + 7) / 8 * 8) + 127) >> 7);
  if (tiles < (conv.p.M <= 64 ? 512 : g.HW % 8 != 0 ? 120 : 257)) return -1;
  const double batched = g.HW >= 64 ? batched_us(cc.gemm) : 0.0;  // (smaller planes are not predicted: a tile is half padding)
  return batched > 0.0 && images_us(conv, tiles) > 1.08 * batched ? -1 : c;
}
Problem images_problem(const Problem& conv) {
  Problem pr = conv;
  ConvGeom& g = pr.p.g;
  pr.images = 1;
  g.H = g.OH = 1;
  g.W = g.OW = g.HW;
  g.OWP = (g.HW + 7) / 8 * 8;
  g.d_owp = make_fastdiv(g.OWP);
  g.d_oh = make_fastdiv(1);
  pr.p.N = (int)(conv.Nb * g.OWP);
  return pr;
}

hidet_status_t make_conv_call(ConvCall& cc, int in, int out, long long Nb, long long IC, long long H, long long W,
                              long long OC, long long KH, long long KW, long long sh, long long sw, long long ph,
                              long long pw, const void* x, const void* w, void* y, const hidet_epilogue_t* epi) {
  const hidet_status_t st = make_conv_problem(cc.conv, in, out, Nb, IC, H, W, OC, KH, KW, sh, sw, ph, pw, x, w, y, epi);
  if (st != HIDET_OK) return st;
  cc.pointwise = false;
  if (KH == 1 && KW == 1 && sh == 1 && sw == 1 && ph == 0 && pw == 0) {
    hidet_epilogue_t e;
    const hidet_epilogue_t* ep = nullptr;
    if (epi) {  // the residual is a dense tensor of y's shape
      e = *epi;
      e.ld_residual = H * W;
      e.batch_stride_residual = OC * H * W;
      ep = &e;
    }
    cc.pointwise = make_gemm_problem(cc.gemm, in, out, 0, 0, Nb, OC, H * W, IC, w, IC, 0, x, H * W, IC * H * W, y, H * W,
                                     OC * H * W, ep) == HIDET_OK;
    // the activation operand is x here too: the B operand of this GEMM
    cc.gemm.p.relu_b = cc.gemm.p.relu_a;
    cc.gemm.p.relu_a = 0;
  }
  return HIDET_OK;
}

// 3x3 and 5x5 convolutions of unit stride that keep the size, in 16-bit types, from OIHW weights, run from a patch of the input
// in LDS (conv_patch.hip): whole stages of 16 channels, and rows whose border the 256 pixels of a patch hold.
bool patch_form(const Problem& conv, const SplitK& sk) {
  const ConvGeom& g = conv.p.g;
  if (conv.op != 1 || conv.dtype == HIDET_F32 || conv.packed || conv.elem_mode != 0) return false;
  if (conv.p.relu_b != 0 || sk.slices > 1) return false;
  if (g.KH != g.KW || (g.KW != 3 && g.KW != 5) || g.sh != 1 || g.sw != 1 || g.ph != g.KH / 2 || g.pw != g.KW / 2) return false;
  if (g.IC % 16 != 0 || g.IC == 0 || conv.p.M == 0 || conv.Nb == 0 || g.W > (g.KW == 3 ? 62 : 29) || g.HW < 8) return false;
  return sat_mul(conv.Nb, (long long)(g.H + g.ph) * (g.W + g.pw)) <= kMaxDim;
}
// Microseconds of a convolution through the gather on the tile that would be taken, and from a patch: predictions for the choice
// between the two alone.  A tile that owns a compute unit (schedules 1 and 3) takes a fixed time and a rate per value of K for
// each round of 256 workgroups, several that share one as much for what they are of a round; a patch a rate per stage and per
// store of its outputs.  Fitted to 2600 random convolutions of 16 to 1024 channels and planes of 6x6 to 62x62, patches of 5x5
// to 400 (relative): 5 % to 95 % of predictions over measurements 0.91 to 1.07 for the K-splitting tiles, 0.84 to 1.15 for the
// others, 0.94 to 1.04 and 0.81 to 1.09 for patches of 5x5 and 3x3.
struct GatherTime {
  int bm, bn, sched;  // (0: schedules 0 and 2)
  double fixed, per_k;  // us; of 4608 values of K
};
constexpr GatherTime kGatherTimes[] = {
    {16, 16, 3, 5.5, 11},   {32, 16, 3, 5.5, 11.5}, {16, 32, 3, 5.5, 11.5}, {32, 32, 3, 5.5, 13}, {64, 32, 3, 6, 16},
    {64, 64, 3, 7.5, 28},   {128, 64, 3, 10.5, 34}, {128, 128, 3, 10, 58.5}, {128, 128, 1, 14, 80}, {256, 128, 1, 26, 112},
    {128, 256, 1, 28, 140}, {256, 256, 1, 30, 220}, {16, 64, 0, 11, 41},    {32, 32, 0, 6, 17.5}, {64, 32, 0, 6.5, 19.5},
    {32, 64, 0, 8, 26},     {64, 64, 0, 7, 33},     {128, 64, 0, 10, 42},   {64, 128, 0, 10.5, 67}};
double gather_us(const Problem& conv) {
  const int c = default_config(conv);
  if (c < 0) return 0.0;
  const ConfigRow& r = kConfigs[c];
  const long long tiles = sat_mul((conv.p.M + r.bm - 1) / r.bm, (conv.p.N + r.bn - 1) / r.bn);
  const double rounds = r.sched == 1 || r.sched == 3 ? (double)((tiles + 255) >> 8) : std::max(1.0, (double)tiles / 256.0);
  for (const GatherTime& t : kGatherTimes)
    if (t.bm == r.bm && t.bn == r.bn && t.sched == (r.sched == 2 ? 0 : r.sched))
      return t.fixed + t.per_k * rounds * conv.p.K / 4608.0;
  return 0.0;
}
double patch_us(const Problem& conv, int rows) {
  const ConvGeom& g = conv.p.g;
  const long long tiles_m = (conv.p.M + rows - 1) / rows, columns = conv.Nb * (g.H + g.ph) * (g.W + g.pw);
  const long long tiles = sat_mul(tiles_m, (columns + 127) >> 7);
  const double stages = g.IC / 16, whole = (double)((tiles + 255) >> 8);
  const bool residual = conv.p.residual != nullptr;
  if (g.KW == 3 && rows == 64) return 4.0 + std::max(1.0, (double)tiles / 256.0) * (2.3 + (residual ? 0.8 : 0.0) + 0.75 * stages);
  if (g.KW == 3) return 1.5 + whole * (5.2 + (residual ? 1.4 : 0.0) + 1.07 * stages);
  return 0.2 + whole * (6.1 + (residual ? 1.2 : 0.0) + 1.6 * stages);
}
// Whether they are the better choice, and on tiles of how many rows; 0: the gather is.
// It wants 72 tiles of 64x128 (of columns with the zero columns and rows among them).  Over 130 random problems of 16 to 512
// channels its time over the gather's is 0.75 to 0.87 from 76 to 88 tiles, 0.42 to 0.9 beyond (1.03 once), but 1.1 to 1.3 from
// 44 to 64, where the gather's K-splitting tiles have twice the workgroups; 58 to 63 tiles of a long K, 0.75 to 0.8, are not
// told from those.  The zeros are no more than two fifths of the outputs (images of 6x6: 1.36 times as many columns, 0.94 to
// 1.07 of the gather's).
// 5x5: 64 rows only, one workgroup to a compute unit, and rows of 29 at most.  From 40 tiles on the predictions decide: over
// 450 random layers of 24 to 1200 tiles this takes 1.005 times as long as the better form of each, 0.84 of the gather's time; 4 are
// more than 4 % slower than the gather (242 of 48x16x16, 32 channels, with residual: 28.3 and 32.6 us).  From fewer tiles on a patch
// is predicted to win only where the two are level (30 of 16x8x8, 368 channels: 7.4 us both).
// 128 rows fetch the input half as often and win from the point where 64 rows are more than one to a compute unit (26 images
// of 128x28x28: 14.7 us, 16.9 us on 64; at most 256 tiles of 64: 1.25 of the time of 64), unless they make a second round
// that is less than half full (47 of 96x27x27, 80 channels, 288 tiles: 23.1 and 21.0 us; 60 of 96x30x30, 451: 26.8 and 29.0
// us; beyond two rounds the two are level, or 64 ahead: 44 of 192x23x23, 384 channels: 57.7 and 55.7 us).
// The counts know neither how many of the gather's columns are padding (none in rows of 8 or 16) nor which tiles it has: where
// the predictions say that it is faster it is taken.  Of 2600 random convolutions 136 were more than 4 % slower than through it
// by the counts alone (13 of 512x8x8, 3x3: 22 and 28 us), 16 are now, none by more than a quarter (154 of 96x8x8, 384 channels,
// 3x3, with residual: 20.9 and 25.8 us).
int patch_rows(const Problem& conv, const SplitK& sk) {
  const ConvGeom& g = conv.p.g;
  if (!patch_form(conv, sk) || conv.p.M < 16) return 0;
  const long long plane = (long long)(g.H + g.ph) * (g.W + g.pw);
  if (5 * plane > (g.KW == 3 ? 7 : 9) * (long long)g.HW) return 0;
  const long long across = (conv.Nb * plane + 127) >> 7;
  const long long of_64 = ((conv.p.M + 63LL) >> 6) * across, of_128 = ((conv.p.M + 127LL) >> 7) * across;
  if (of_64 < (g.KW == 3 ? 72 : 40)) return 0;
  const int rows = g.KW == 3 && conv.p.M > 64 && of_64 > 256 && (of_128 <= 256 || (of_128 > 384 && of_128 <= 512)) ? 128 : 64;
  const double gather = gather_us(conv);
  return gather > 0.0 && patch_us(conv, rows) > gather * 1.05 ? 0 : rows;
}
hidet_status_t launch_patch(const Problem& conv, int bm, hipStream_t stream) {
  GemmParams p = conv.p;
  const int zeros = p.g.KW / 2;
  p.g.d_owp = make_fastdiv(p.g.W + zeros);
  p.g.d_oh = make_fastdiv(p.g.H + zeros);
  p.N = (int)(conv.Nb * (p.g.H + zeros) * (p.g.W + zeros));
  const int tiles_m = (p.M + bm - 1) / bm, tiles_n = (p.N + 127) / 128;
  set_block_mapping(p, tiles_m, tiles_n, tiles_m >= 4 ? 4 : tiles_m);
  p.k_slices = 1;
  p.k_slice_len = p.K;
  const long long total = (long long)tiles_m * tiles_n;
  if (total > kIntMax) return HIDET_ERR_UNSUPPORTED;
  p.total_blocks = (int)total;
  const hipError_t e = conv.dtype == HIDET_F16 ? launch_conv_patch_f16(p, bm, stream) : launch_conv_patch_bf16(p, bm, stream);
  if (e != hipSuccess) return HIDET_ERR_LAUNCH;
  ++g_kernel_launches;
  return HIDET_OK;
}

// One form of a convolution; a form that cannot run the call is refused before anything is launched.
hidet_status_t launch_form(const ConvCall& cc, int form, int config, const SplitK& sk, hipStream_t stream) {
  switch (form) {
    case HIDET_CONV_GATHER: return launch(cc.conv, config, sk, stream);
    case HIDET_CONV_BATCHED: return cc.pointwise ? launch(cc.gemm, config, sk, stream) : HIDET_ERR_NO_CONFIG;
    case HIDET_CONV_IMAGES:
      if (images_form(cc.conv, cc.pointwise, sk) < 0) return HIDET_ERR_NO_CONFIG;
      return launch(images_problem(cc.conv), config, SplitK(), stream);
    case HIDET_CONV_PATCH_64:
    case HIDET_CONV_PATCH_128:
      if (!patch_form(cc.conv, sk) || (form == HIDET_CONV_PATCH_128 && cc.conv.p.g.KW != 3)) return HIDET_ERR_NO_CONFIG;
      return launch_patch(cc.conv, form == HIDET_CONV_PATCH_64 ? 64 : 128, stream);
    default: return HIDET_ERR_NO_CONFIG;
  }
}

// What a call runs that names no configuration and for which nothing is remembered.
int untuned_form(const ConvCall& cc, const SplitK& sk) {
  const int rows = patch_rows(cc.conv, sk);
  if (rows > 0) return rows == 64 ? HIDET_CONV_PATCH_64 : HIDET_CONV_PATCH_128;
  if (!cc.pointwise) return HIDET_CONV_GATHER;
  return images_config(cc, sk) >= 0 ? HIDET_CONV_IMAGES : HIDET_CONV_BATCHED;
}

// An explicit configuration always runs the gather form; config < 0 runs what the tuner remembered for this
// convolution, else (3x3 and 5x5 convolutions) the patch kernel or (1x1 convolutions) the product over all images or the
// batched-GEMM form with its size-based default.
hidet_status_t launch_conv(const ConvCall& cc, int config, const SplitK& sk, hipStream_t stream) {
  if (config >= 0 || (!cc.pointwise && !patch_form(cc.conv, sk))) return launch(cc.conv, config, sk, stream);
  Tuned t{-1, 1, HIDET_CONV_GATHER};
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    auto it = find_tuned(cc.conv, sk);
    if (it != g_cache.end()) t = it->second;
  }
  SplitK one = sk;
  if (one.slices < 0) one.slices = t.slices;
  // (an entry that cannot serve this call -- more K slices than the remembered form has, a file written elsewhere -- counts for
  // the configuration of the gather where it is one, else as if nothing were remembered)
  if (t.config >= 0 && t.form >= HIDET_CONV_IMAGES) {
    const hidet_status_t st = launch_form(cc, t.form, t.config, sk, stream);
    if (st != HIDET_ERR_NO_CONFIG) return st;
  }
  const Problem& remembered = t.form == HIDET_CONV_BATCHED && cc.pointwise ? cc.gemm : cc.conv;
  if (t.form != HIDET_CONV_IMAGES && find_launcher(remembered, t.config) &&
      (one.slices <= 1 || find_partial_launcher(remembered, t.config)))
    return launch(remembered, t.config, one, stream);
  const int form = untuned_form(cc, sk);
  const int c = form == HIDET_CONV_GATHER   ? default_config(cc.conv)
                : form == HIDET_CONV_IMAGES ? images_form(cc.conv, cc.pointwise, sk)
                                            : -1;
  return launch_form(cc, form, c, sk, stream);
}

// Tunes the gather and whatever other forms can run the call -- the batched GEMM and the product over all images of a 1x1
// convolution, the patch of a 3x3 or 5x5 one; the fastest is remembered under the convolution's key.
hidet_status_t tune_conv(const ConvCall& cc, const SplitK& sk, hipStream_t stream, int iters, int32_t* best_config,
                         int32_t* best_slices, float* best_us) {
  int32_t c0 = -1, s0 = 1;
  float t0 = 0.0f;
  int form = HIDET_CONV_GATHER;
  hidet_status_t st = tune(cc.conv, sk, stream, iters, &c0, &s0, &t0);
  if (st != HIDET_OK) return st;
  if (cc.pointwise) {
    std::vector<float> times0;
    {
      std::lock_guard<std::mutex> lock(g_mutex);
      times0 = g_last_times;
    }
    int32_t c1 = -1, s1 = 1;
    float t1 = 0.0f;
    st = tune(cc.gemm, sk, stream, iters, &c1, &s1, &t1);
    if (st != HIDET_OK) return st;
    std::lock_guard<std::mutex> lock(g_mutex);
    for (size_t i = 0; i < g_last_times.size() && i < times0.size(); ++i)
      if (times0[i] >= 0.0f && (g_last_times[i] < 0.0f || times0[i] < g_last_times[i])) g_last_times[i] = times0[i];
    if (c1 >= 0 && (c0 < 0 || t1 < t0)) {
      form = HIDET_CONV_BATCHED;
      c0 = c1;
      s0 = s1;
      t0 = t1;
    }
  }
  if (c0 >= 0) {
    const SplitK whole;
    const int images = images_form(cc.conv, cc.pointwise, whole);
    Stopwatch watch(stream, iters);
    if (!watch.ready()) return HIDET_ERR_LAUNCH;
    for (int f : {HIDET_CONV_IMAGES, HIDET_CONV_PATCH_64, HIDET_CONV_PATCH_128}) {
      float us = 0.0f;
      if (!watch.time([&] { return launch_form(cc, f, images, whole, stream); }, &us)) return HIDET_ERR_LAUNCH;
      if (us < 0.0f) continue;
      std::lock_guard<std::mutex> lock(g_mutex);
      if (f == HIDET_CONV_IMAGES && (g_last_times[images] < 0.0f || us < g_last_times[images])) g_last_times[images] = us;
      if (us >= t0) continue;
      form = f;
      t0 = us;
      if (f == HIDET_CONV_IMAGES) {
        c0 = images;
        s0 = 1;
      }
    }
    SplitK win = form <= HIDET_CONV_BATCHED ? sk : whole;  // (the winner's output is left in the buffer)
    if (form <= HIDET_CONV_BATCHED) win.slices = s0;
    launch_form(cc, form, c0, win, stream);
    (void)hipStreamSynchronize(stream);
    std::lock_guard<std::mutex> lock(g_mutex);
    g_cache[problem_key(cc.conv, sk.workspace != nullptr)] = Tuned{c0, s0, form};
  }
  if (best_config) *best_config = c0;
  if (best_slices) *best_slices = s0;
  if (best_us) *best_us = t0;
  return HIDET_OK;
}

// ---- convolution with repacked weights ----------------------------------------------------------------------------
// OIHW -> O(HW)I: w_packed[oc][kh][kw][ic] = w[oc][ic][kh][kw].  With the K axis of the implicit GEMM ordered
// (kh, kw, ic) a K tile lies within one filter tap, which makes the padding mask and the spatial offset of the img2col
// gather the same for all of a thread's chunks of the tile (Operand::request_tile).
template <typename U>
__global__ void __launch_bounds__(256) pack_weights_kernel(const U* __restrict__ w, U* __restrict__ wp, long long total,
                                                          int IC, int KHW, FastDiv d_ic) {
  const long long o = (long long)blockIdx.x * 256 + threadIdx.x;
  if (o >= total) return;
  // o = (oc * KHW + t) * IC + ic; rows of KHW * IC elements stay below 2^31 (checked on the host)
  const long long row = o / ((long long)KHW * IC);
  const int in_row = (int)(o - row * ((long long)KHW * IC));
  const int t = d_ic.div(in_row), ic = in_row - t * IC;
  wp[o] = w[row * ((long long)KHW * IC) + (long long)ic * KHW + t];
}

// The packed form: a ConvCall whose gather problem is marked `packed`.  Needs IC % 8 == 0 (16-byte rows of the
// repacked weights), strides of at most 2 and an input of at least two chunks.
hidet_status_t make_packed_conv_call(ConvCall& cc, int in, int out, long long Nb, long long IC, long long H, long long W,
                                     long long OC, long long KH, long long KW, long long sh, long long sw, long long ph,
                                     long long pw, const void* x, const void* w_packed, void* y,
                                     const hidet_epilogue_t* epi) {
  const hidet_status_t st = make_conv_problem(cc.conv, in, out, Nb, IC, H, W, OC, KH, KW, sh, sw, ph, pw, x, w_packed, y, epi);
  if (st != HIDET_OK) return st;
  const int vec = 16 / elem_size(in);
  if (IC % vec != 0 || sw > 2 || Nb * IC * H * W < 4 * vec || cc.conv.elem_mode != 0) return HIDET_ERR_UNSUPPORTED;
  cc.conv.packed = 1;
  cc.pointwise = false;
  return HIDET_OK;
}

// ---- task-mapping instances exposed to tests ----------------------------------------------------------
struct TaskMapEntry {
  const char* expr;
  int workers, shape0, shape1, tasks;
  tmap::Task (*task)(int, int);
};
template <class M>
TaskMapEntry tm_entry(const char* expr) {
  return TaskMapEntry{expr, M::workers, M::shape0, M::shape1, M::tasks, [](int w, int q) { return M::task(w, q); }};
}
using namespace hidet::tmap;
const TaskMapEntry kTaskMaps[] = {
    // the paper's worked examples
    tm_entry<Compose<Repeat<4, 1>, Spatial<16, 8>>>("repeat(4,1)*spatial(16,8)"),
    tm_entry<Chain<Spatial<4, 2>, Repeat<2, 2>, Spatial<4, 8>, Repeat<4, 4>>>(
        "spatial(4,2)*repeat(2,2)*spatial(4,8)*repeat(4,4)"),
    tm_entry<Compose<Spatial<2, 2>, Repeat<2, 2>>>("spatial(2,2)*repeat(2,2)"),
    tm_entry<Repeat<2, 2>>("repeat(2,2)"),
    tm_entry<Spatial<2, 2>>("spatial(2,2)"),
    tm_entry<Compose<Spatial<1, 3>, Spatial<2, 1>>>("spatial(1,3)*spatial(2,1)"),
    tm_entry<Compose<Compose<Repeat<2, 1>, Spatial<2, 3>>, Repeat<1, 2>>>("repeat(2,1)*spatial(2,3)*repeat(1,2)"),
    tm_entry<Compose<Repeat<2, 1>, Compose<Spatial<2, 3>, Repeat<1, 2>>>>("repeat(2,1)*spatial(2,3)*repeat(1,2)"),
    // the mappings the headline kernel (configuration 19: 256x256x32 tile, 8 waves, 16x16x32 matrix-core tiles) walks:
    // its direct global -> LDS loads (Operand::init_direct) and its wave -> MFMA-tile assignment
    tm_entry<LoadMapRowMajor<256, 4, 512>::Map>("repeat(2,1)*spatial(128,4)"),   // A tile, 256 rows x 4 chunks
    tm_entry<LoadMapRowMajor<32, 32, 512>::Map>("repeat(2,1)*spatial(16,32)"),   // B tile, 32 k-rows x 32 chunks
    tm_entry<Compose<Spatial<2, 4>, Repeat<8, 4>>>("spatial(2,4)*repeat(8,4)"),  // waves -> MFMA tiles
    // the same for the general schedule on a 256x256x64 tile with 32x32x16 tiles (configuration 20)
    tm_entry<LoadMapRowMajor<256, 8, 512>::Map>("repeat(4,1)*spatial(64,8)"),    // A tile, 256 rows x 8 chunks
    tm_entry<LoadMapRowMajor<64, 32, 512>::Map>("repeat(4,1)*spatial(16,32)"),   // B tile, 64 k-rows x 32 chunks
    tm_entry<Compose<Spatial<2, 4>, Repeat<4, 2>>>("spatial(2,4)*repeat(4,2)"),  // waves -> MFMA tiles
    // fp32 A tile of the 128x128x16 configuration: threads walk down the rows first
    tm_entry<LoadMapColMajor<128, 4, 256>::Map>("repeat(2,1)*spatial(2,128)"),
    tm_entry<LoadMapColMajor<256, 4, 128>::Map>("repeat(4,2)*spatial(1,128)"),
};
const int kNumTaskMaps = (int)(sizeof(kTaskMaps) / sizeof(kTaskMaps[0]));

}  // namespace

// ------------------------------------------------------------------------------------------------
// exported functions
// ------------------------------------------------------------------------------------------------
extern "C" {

hidet_status_t hidet_batched_gemm_cfg(int32_t config, int32_t in, int32_t out, int32_t transA, int32_t transB,
                                      int64_t batch, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
                                      int64_t strideA, const void* B, int64_t ldb, int64_t strideB, void* C,
                                      int64_t ldc, int64_t strideC, const hidet_epilogue_t* epi, void* stream) {
  Problem pr;
  hidet_status_t st = make_gemm_problem(pr, in, out, transA, transB, batch, M, N, K, A, lda, strideA, B, ldb, strideB,
                                        C, ldc, strideC, epi);
  if (st != HIDET_OK) return st;
  if (config >= kNumConfigs) return HIDET_ERR_NO_CONFIG;
  return guarded([&] { return launch(pr, config, SplitK{}, (hipStream_t)stream); });
}

hidet_status_t hidet_gemm_cfg(int32_t config, int32_t in, int32_t out, int32_t transA, int32_t transB, int64_t M,
                              int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb, void* C,
                              int64_t ldc, const hidet_epilogue_t* epi, void* stream) {
  return hidet_batched_gemm_cfg(config, in, out, transA, transB, 1, M, N, K, A, lda, 0, B, ldb, 0, C, ldc, 0, epi,
                                stream);
}

hidet_status_t hidet_gemm(int32_t in, int32_t out, int32_t transA, int32_t transB, int64_t M, int64_t N, int64_t K,
                          const void* A, int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc,
                          const hidet_epilogue_t* epi, void* stream) {
  return hidet_gemm_cfg(-1, in, out, transA, transB, M, N, K, A, lda, B, ldb, C, ldc, epi, stream);
}

hidet_status_t hidet_batched_gemm(int32_t in, int32_t out, int32_t transA, int32_t transB, int64_t batch, int64_t M,
                                  int64_t N, int64_t K, const void* A, int64_t lda, int64_t strideA, const void* B,
                                  int64_t ldb, int64_t strideB, void* C, int64_t ldc, int64_t strideC,
                                  const hidet_epilogue_t* epi, void* stream) {
  return hidet_batched_gemm_cfg(-1, in, out, transA, transB, batch, M, N, K, A, lda, strideA, B, ldb, strideB, C, ldc,
                                strideC, epi, stream);
}

hidet_status_t hidet_conv2d_implicit_gemm_cfg(int32_t config, int32_t in, int32_t out, int64_t Nb, int64_t IC,
                                              int64_t H, int64_t W, int64_t OC, int64_t KH, int64_t KW,
                                              int64_t stride_h, int64_t stride_w, int64_t pad_h, int64_t pad_w,
                                              const void* x, const void* w, void* y, const hidet_epilogue_t* epi,
                                              void* stream) {
  ConvCall cc;
  hidet_status_t st = make_conv_call(cc, in, out, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h, pad_w, x, w, y,
                                     epi);
  if (st != HIDET_OK) return st;
  if (config >= kNumConfigs) return HIDET_ERR_NO_CONFIG;
  return guarded([&] { return launch_conv(cc, config, SplitK{}, (hipStream_t)stream); });
}

hidet_status_t hidet_conv2d_implicit_gemm(int32_t in, int32_t out, int64_t Nb, int64_t IC, int64_t H, int64_t W,
                                          int64_t OC, int64_t KH, int64_t KW, int64_t stride_h, int64_t stride_w,
                                          int64_t pad_h, int64_t pad_w, const void* x, const void* w, void* y,
                                          const hidet_epilogue_t* epi, void* stream) {
  return hidet_conv2d_implicit_gemm_cfg(-1, in, out, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h, pad_w, x, w,
                                        y, epi, stream);
}

int32_t hidet_config_count(void) { return kNumConfigs; }

hidet_status_t hidet_config_info(int32_t config, hidet_config_info_t* info) {
  if (!info) return HIDET_ERR_INVALID_ARG;
  if (config < 0 || config >= kNumConfigs) return HIDET_ERR_NO_CONFIG;
  const ConfigRow& r = kConfigs[config];
  info->block_m = r.bm;
  info->block_n = r.bn;
  info->block_k = r.bk;
  info->waves_m = r.waves_m;
  info->waves_n = r.waves_n;
  info->mfma = r.mfma;
  info->is_f32 = r.is_f32;
  info->schedule = r.sched;
  info->stages = r.sched == 1 ? 4 : 2;
  info->waves_k = r.sched == 3 ? 16 / (r.waves_m * r.waves_n) : 1;
  const int staging = info->stages * (r.bm + r.bn) * r.bk * (r.is_f32 ? 4 : 2);
  int epilogue = r.waves_m * r.mfma * (r.bn * 4 + 16 * r.waves_n);  // per-wave transposition regions
  if (r.sched == 3) epilogue += (16 / (r.waves_m * r.waves_n) - 1) * r.bm * r.bn * 4;  // partial sums of the wave groups along K
  // (of K tiles that all wavefronts share, also for the tiles of schedule 3 whose GEMMs have wavefronts that share nothing; a
  // convolution adds a 1.3 KB mask table)
  info->lds_bytes = staging > epilogue ? staging : epilogue;
  return HIDET_OK;
}

hidet_status_t hidet_tune_gemm(int32_t in, int32_t out, int32_t transA, int32_t transB, int64_t batch, int64_t M,
                               int64_t N, int64_t K, const void* A, int64_t lda, int64_t strideA, const void* B,
                               int64_t ldb, int64_t strideB, void* C, int64_t ldc, int64_t strideC,
                               const hidet_epilogue_t* epi, void* stream, int32_t iters, int32_t* best_config,
                               float* best_us) {
  Problem pr;
  hidet_status_t st = make_gemm_problem(pr, in, out, transA, transB, batch, M, N, K, A, lda, strideA, B, ldb, strideB,
                                        C, ldc, strideC, epi);
  if (st != HIDET_OK) return st;
  return guarded([&] { return tune(pr, SplitK{}, (hipStream_t)stream, iters, best_config, nullptr, best_us); });
}

hidet_status_t hidet_tune_conv2d(int32_t in, int32_t out, int64_t Nb, int64_t IC, int64_t H, int64_t W, int64_t OC,
                                 int64_t KH, int64_t KW, int64_t stride_h, int64_t stride_w, int64_t pad_h,
                                 int64_t pad_w, const void* x, const void* w, void* y, const hidet_epilogue_t* epi,
                                 void* stream, int32_t iters, int32_t* best_config, float* best_us) {
  ConvCall cc;
  hidet_status_t st = make_conv_call(cc, in, out, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h, pad_w, x, w, y,
                                     epi);
  if (st != HIDET_OK) return st;
  return guarded([&] { return tune_conv(cc, SplitK{}, (hipStream_t)stream, iters, best_config, nullptr, best_us); });
}

// ---- K-parallel ("split-K") forms ------------------------------------------------------------------------------
int64_t hidet_splitk_workspace_bytes(int64_t batch, int64_t M, int64_t N, int32_t k_slices) {
  if (batch < 0 || M < 0 || N < 0 || k_slices < 1) return -1;
  const long long bytes = sat_mul(sat_mul(sat_mul(4LL * k_slices, batch), M), N);
  return bytes >= (1LL << 62) ? -1 : bytes;
}

hidet_status_t hidet_batched_gemm_splitk(int32_t config, int32_t k_slices, int32_t in, int32_t out, int32_t transA,
                                         int32_t transB, int64_t batch, int64_t M, int64_t N, int64_t K, const void* A,
                                         int64_t lda, int64_t strideA, const void* B, int64_t ldb, int64_t strideB,
                                         void* C, int64_t ldc, int64_t strideC, const hidet_epilogue_t* epi,
                                         void* workspace, int64_t workspace_bytes, void* stream) {
  Problem pr;
  hidet_status_t st = make_gemm_problem(pr, in, out, transA, transB, batch, M, N, K, A, lda, strideA, B, ldb, strideB,
                                        C, ldc, strideC, epi);
  if (st != HIDET_OK) return st;
  if (config >= kNumConfigs) return HIDET_ERR_NO_CONFIG;
  if (workspace_bytes < 0 || k_slices > 1024) return HIDET_ERR_INVALID_ARG;
  SplitK sk;
  sk.slices = k_slices <= 0 ? -1 : k_slices;
  sk.workspace = workspace;
  sk.workspace_bytes = workspace_bytes;
  return guarded([&] { return launch(pr, config, sk, (hipStream_t)stream); });
}

hidet_status_t hidet_conv2d_implicit_gemm_splitk(int32_t config, int32_t k_slices, int32_t in, int32_t out, int64_t Nb,
                                                 int64_t IC, int64_t H, int64_t W, int64_t OC, int64_t KH, int64_t KW,
                                                 int64_t stride_h, int64_t stride_w, int64_t pad_h, int64_t pad_w,
                                                 const void* x, const void* w, void* y, const hidet_epilogue_t* epi,
                                                 void* workspace, int64_t workspace_bytes, void* stream) {
  ConvCall cc;
  hidet_status_t st = make_conv_call(cc, in, out, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h, pad_w, x, w, y,
                                     epi);
  if (st != HIDET_OK) return st;
  if (config >= kNumConfigs) return HIDET_ERR_NO_CONFIG;
  if (workspace_bytes < 0 || k_slices > 1024) return HIDET_ERR_INVALID_ARG;
  SplitK sk;
  sk.slices = k_slices <= 0 ? -1 : k_slices;
  sk.workspace = workspace;
  sk.workspace_bytes = workspace_bytes;
  return guarded([&] { return launch_conv(cc, config, sk, (hipStream_t)stream); });
}

hidet_status_t hidet_conv2d_pack_weights(int32_t dtype, int64_t OC, int64_t IC, int64_t KH, int64_t KW, const void* w,
                                         void* w_packed, void* stream) {
  if (dtype < 0 || dtype > 2 || OC < 0 || IC < 0 || KH <= 0 || KW <= 0) return HIDET_ERR_INVALID_ARG;
  if (KH > 32767 || KW > 32767 || IC > kMaxDim || OC > kMaxDim || sat_mul(IC, KH * KW) > kMaxDim) return HIDET_ERR_UNSUPPORTED;
  const long long total = sat_mul(OC, IC * KH * KW);
  if (total == 0) return HIDET_OK;
  if (total > (1LL << 40)) return HIDET_ERR_UNSUPPORTED;
  if (!w || !w_packed) return HIDET_ERR_INVALID_ARG;
  const size_t es = (size_t)elem_size(dtype);
  if (!aligned(w, es) || !aligned(w_packed, es)) return HIDET_ERR_ALIGNMENT;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  if (es == 2)
    hipLaunchKernelGGL(pack_weights_kernel<unsigned short>, dim3(blocks), dim3(256), 0, (hipStream_t)stream,
                       (const unsigned short*)w, (unsigned short*)w_packed, total, (int)IC, (int)(KH * KW), make_fastdiv(IC));
  else
    hipLaunchKernelGGL(pack_weights_kernel<unsigned int>, dim3(blocks), dim3(256), 0, (hipStream_t)stream,
                       (const unsigned int*)w, (unsigned int*)w_packed, total, (int)IC, (int)(KH * KW), make_fastdiv(IC));
  return hipGetLastError() == hipSuccess ? HIDET_OK : HIDET_ERR_LAUNCH;
}

hidet_status_t hidet_conv2d_implicit_gemm_packed(int32_t config, int32_t k_slices, int32_t in, int32_t out, int64_t Nb,
                                                 int64_t IC, int64_t H, int64_t W, int64_t OC, int64_t KH, int64_t KW,
                                                 int64_t stride_h, int64_t stride_w, int64_t pad_h, int64_t pad_w,
                                                 const void* x, const void* w_packed, void* y, const hidet_epilogue_t* epi,
                                                 void* workspace, int64_t workspace_bytes, void* stream) {
  ConvCall cc;
  hidet_status_t st = make_packed_conv_call(cc, in, out, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h, pad_w, x,
                                            w_packed, y, epi);
  if (st != HIDET_OK) return st;
  if (config >= kNumConfigs) return HIDET_ERR_NO_CONFIG;
  if (workspace_bytes < 0 || k_slices > 1024) return HIDET_ERR_INVALID_ARG;
  SplitK sk;
  sk.slices = k_slices <= 0 ? (workspace ? -1 : 1) : k_slices;
  sk.workspace = workspace;
  sk.workspace_bytes = workspace_bytes;
  return guarded([&] { return launch(cc.conv, config, sk, (hipStream_t)stream); });
}

hidet_status_t hidet_tune_conv2d_packed(int32_t in, int32_t out, int64_t Nb, int64_t IC, int64_t H, int64_t W, int64_t OC,
                                        int64_t KH, int64_t KW, int64_t stride_h, int64_t stride_w, int64_t pad_h,
                                        int64_t pad_w, const void* x, const void* w_packed, void* y,
                                        const hidet_epilogue_t* epi, void* workspace, int64_t workspace_bytes, void* stream,
                                        int32_t iters, int32_t* best_config, int32_t* best_slices, float* best_us) {
  ConvCall cc;
  hidet_status_t st = make_packed_conv_call(cc, in, out, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h, pad_w, x,
                                            w_packed, y, epi);
  if (st != HIDET_OK) return st;
  if (workspace_bytes < 0) return HIDET_ERR_INVALID_ARG;
  SplitK sk;
  sk.workspace = workspace;
  sk.workspace_bytes = workspace ? workspace_bytes : 0;
  return guarded([&] { return tune(cc.conv, sk, (hipStream_t)stream, iters, best_config, best_slices, best_us); });
}

hidet_status_t hidet_conv2d_untuned_config(int32_t in, int64_t Nb, int64_t IC, int64_t H, int64_t W, int64_t OC, int64_t KH,
                                           int64_t KW, int64_t stride_h, int64_t stride_w, int64_t pad_h, int64_t pad_w,
                                           int32_t packed, int32_t* config) {
  if (!config) return HIDET_ERR_INVALID_ARG;
  // (16-byte aligned stand-ins for the tensors: the choice looks at their alignment alone)
  void* const at = reinterpret_cast<void*>((uintptr_t)4096);
  ConvCall cc;
  const hidet_status_t st = packed ? make_packed_conv_call(cc, in, in, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h,
                                                           pad_w, at, at, at, nullptr)
                                   : make_conv_call(cc, in, in, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h, pad_w,
                                                    at, at, at, nullptr);
  if (st != HIDET_OK) return st;
  const Problem& pr = cc.pointwise ? cc.gemm : cc.conv;
  const int images = images_config(cc, SplitK());
  *config = images >= 0 ? images : pr.batch == 0 || pr.p.M == 0 || pr.p.N == 0 ? -1 : default_config(pr);
  return HIDET_OK;
}

hidet_status_t hidet_conv2d_untuned_form(int32_t in, int64_t Nb, int64_t IC, int64_t H, int64_t W, int64_t OC, int64_t KH, int64_t KW,
                                         int64_t stride_h, int64_t stride_w, int64_t pad_h, int64_t pad_w, int32_t* form) {
  if (!form) return HIDET_ERR_INVALID_ARG;
  void* const at = reinterpret_cast<void*>((uintptr_t)4096);  // (as above)
  ConvCall cc;
  const hidet_status_t st =
      make_conv_call(cc, in, in, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h, pad_w, at, at, at, nullptr);
  if (st != HIDET_OK) return st;
  *form = cc.conv.p.M == 0 || cc.conv.p.N == 0 ? -1 : untuned_form(cc, SplitK());
  return HIDET_OK;
}

hidet_status_t hidet_conv2d_patch_rows(int32_t in, int64_t Nb, int64_t IC, int64_t H, int64_t W, int64_t OC, int64_t KH, int64_t KW,
                                       int64_t stride_h, int64_t stride_w, int64_t pad_h, int64_t pad_w, int32_t* rows) {
  if (!rows) return HIDET_ERR_INVALID_ARG;
  void* const at = reinterpret_cast<void*>((uintptr_t)4096);  // (as above)
  ConvCall cc;
  const hidet_status_t st =
      make_conv_call(cc, in, in, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h, pad_w, at, at, at, nullptr);
  if (st != HIDET_OK) return st;
  *rows = patch_rows(cc.conv, SplitK());
  return HIDET_OK;
}

hidet_status_t hidet_gemm_untuned_config(int32_t in, int32_t transA, int32_t transB, int64_t batch, int64_t M, int64_t N,
                                         int64_t K, int32_t* config) {
  if (!config) return HIDET_ERR_INVALID_ARG;
  void* const at = reinterpret_cast<void*>((uintptr_t)4096);  // (as above)
  const long long lda = transA ? M : K, ldb = transB ? K : N;
  Problem pr;
  const hidet_status_t st = make_gemm_problem(pr, in, in, transA, transB, batch, M, N, K, at, lda, sat_mul(M, K), at, ldb,
                                              sat_mul(N, K), at, N, sat_mul(M, N), nullptr);
  if (st != HIDET_OK) return st;
  *config = pr.batch == 0 || pr.p.M == 0 || pr.p.N == 0 ? -1 : default_config(pr);
  return HIDET_OK;
}

int64_t hidet_conv2d_splitk_workspace_bytes(int64_t Nb, int64_t OC, int64_t OH, int64_t OW, int32_t k_slices) {
  if (Nb < 0 || OC < 0 || OH < 0 || OW < 0 || OW > kIntMax) return -1;
  // GEMM columns of the implicit GEMM: every output row padded to a multiple of 8 positions (see ConvGeom)
  return hidet_splitk_workspace_bytes(1, OC, sat_mul(sat_mul(Nb, OH), (OW + 7) / 8 * 8), k_slices);
}

int64_t hidet_static_scratch_bytes(void) { return kScratchBytes; }

hidet_status_t hidet_batched_gemm_splitk_static(int32_t config, int32_t k_slices, int32_t in, int32_t out,
                                                int32_t transA, int32_t transB, int64_t batch, int64_t M, int64_t N,
                                                int64_t K, const void* A, int64_t lda, int64_t strideA, const void* B,
                                                int64_t ldb, int64_t strideB, void* C, int64_t ldc, int64_t strideC,
                                                const hidet_epilogue_t* epi, void* stream) {
  Problem pr;
  hidet_status_t st = make_gemm_problem(pr, in, out, transA, transB, batch, M, N, K, A, lda, strideA, B, ldb, strideB,
                                        C, ldc, strideC, epi);
  if (st != HIDET_OK) return st;
  if (config >= kNumConfigs) return HIDET_ERR_NO_CONFIG;
  if (k_slices > 1024) return HIDET_ERR_INVALID_ARG;
  SplitK sk;
  sk.slices = k_slices <= 0 ? -1 : k_slices;
  sk.workspace_bytes = kScratchBytes;
  sk.fixed = true;
  st = scratch_of_current_device(&sk.workspace);
  if (st != HIDET_OK) return st;
  return guarded([&] { return launch(pr, config, sk, (hipStream_t)stream); });
}

hidet_status_t hidet_tune_gemm_splitk(int32_t in, int32_t out, int32_t transA, int32_t transB, int64_t batch, int64_t M,
                                      int64_t N, int64_t K, const void* A, int64_t lda, int64_t strideA, const void* B,
                                      int64_t ldb, int64_t strideB, void* C, int64_t ldc, int64_t strideC,
                                      const hidet_epilogue_t* epi, void* workspace, int64_t workspace_bytes, void* stream,
                                      int32_t iters, int32_t* best_config, int32_t* best_slices, float* best_us) {
  Problem pr;
  hidet_status_t st = make_gemm_problem(pr, in, out, transA, transB, batch, M, N, K, A, lda, strideA, B, ldb, strideB,
                                        C, ldc, strideC, epi);
  if (st != HIDET_OK) return st;
  if (!workspace || workspace_bytes <= 0) return HIDET_ERR_INVALID_ARG;
  SplitK sk;
  sk.workspace = workspace;
  sk.workspace_bytes = workspace_bytes;
  return guarded([&] { return tune(pr, sk, (hipStream_t)stream, iters, best_config, best_slices, best_us); });
}

hidet_status_t hidet_tune_conv2d_splitk(int32_t in, int32_t out, int64_t Nb, int64_t IC, int64_t H, int64_t W,
                                        int64_t OC, int64_t KH, int64_t KW, int64_t stride_h, int64_t stride_w,
                                        int64_t pad_h, int64_t pad_w, const void* x, const void* w, void* y,
                                        const hidet_epilogue_t* epi, void* workspace, int64_t workspace_bytes,
                                        void* stream, int32_t iters, int32_t* best_config, int32_t* best_slices,
                                        float* best_us) {
  ConvCall cc;
  hidet_status_t st = make_conv_call(cc, in, out, Nb, IC, H, W, OC, KH, KW, stride_h, stride_w, pad_h, pad_w, x, w, y,
                                     epi);
  if (st != HIDET_OK) return st;
  if (!workspace || workspace_bytes <= 0) return HIDET_ERR_INVALID_ARG;
  SplitK sk;
  sk.workspace = workspace;
  sk.workspace_bytes = workspace_bytes;
  return guarded([&] { return tune_conv(cc, sk, (hipStream_t)stream, iters, best_config, best_slices, best_us); });
}

int32_t hidet_tune_last_times(float* us_per_config, int32_t capacity) {
  std::lock_guard<std::mutex> lock(g_mutex);
  const int n = (int)g_last_times.size();
  if (us_per_config)
    for (int i = 0; i < n && i < capacity; ++i) us_per_config[i] = g_last_times[i];
  return n;
}

void hidet_tune_clear(void) {
  std::lock_guard<std::mutex> lock(g_mutex);
  g_cache.clear();
}

hidet_status_t hidet_tune_save(const char* path) {
  if (!path) return HIDET_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lock(g_mutex);
  FILE* f = std::fopen(path, "w");
  if (!f) return HIDET_ERR_INVALID_ARG;
  for (const auto& kv : g_cache)
    std::fprintf(f, "%s %d %d %d\n", kv.first.c_str(), kv.second.config, kv.second.slices, kv.second.form);
  std::fclose(f);
  return HIDET_OK;
}

hidet_status_t hidet_tune_load(const char* path) {
  if (!path) return HIDET_ERR_INVALID_ARG;
  FILE* f = std::fopen(path, "r");
  if (!f) return HIDET_ERR_INVALID_ARG;
  char line[512], key[256];
  const hidet_status_t st = guarded([&] {
    std::lock_guard<std::mutex> lock(g_mutex);
    while (std::fgets(line, sizeof(line), f)) {
      int cfg = 0, slices = 1, form = 0;  // the form is absent from files written before it existed
      if (std::sscanf(line, "%255s %d %d %d", key, &cfg, &slices, &form) < 3) continue;
      if (cfg >= 0 && cfg < kNumConfigs && slices >= 1 && slices <= 1024 && form >= HIDET_CONV_GATHER && form <= HIDET_CONV_PATCH_128)
        g_cache[std::string(key)] = Tuned{cfg, slices, form};
    }
    return HIDET_OK;
  });
  std::fclose(f);
  return st;
}

int32_t hidet_taskmap_count(void) { return kNumTaskMaps; }

hidet_status_t hidet_taskmap_info(int32_t index, char* expr, int32_t expr_capacity, int32_t* workers, int32_t* shape0,
                                  int32_t* shape1, int32_t* tasks_per_worker) {
  if (index < 0 || index >= kNumTaskMaps) return HIDET_ERR_INVALID_ARG;
  const TaskMapEntry& e = kTaskMaps[index];
  if (expr && expr_capacity > 0) {
    std::strncpy(expr, e.expr, (size_t)expr_capacity - 1);
    expr[expr_capacity - 1] = 0;
  }
  if (workers) *workers = e.workers;
  if (shape0) *shape0 = e.shape0;
  if (shape1) *shape1 = e.shape1;
  if (tasks_per_worker) *tasks_per_worker = e.tasks;
  return HIDET_OK;
}

hidet_status_t hidet_taskmap_tasks(int32_t index, int32_t worker, int32_t* tasks_ij, int32_t capacity_pairs) {
  if (index < 0 || index >= kNumTaskMaps || !tasks_ij) return HIDET_ERR_INVALID_ARG;
  const TaskMapEntry& e = kTaskMaps[index];
  if (worker < 0 || worker >= e.workers || capacity_pairs < e.tasks) return HIDET_ERR_INVALID_ARG;
  for (int q = 0; q < e.tasks; ++q) {
    const tmap::Task t = e.task(worker, q);
    tasks_ij[2 * q] = t.i;
    tasks_ij[2 * q + 1] = t.j;
  }
  return HIDET_OK;
}

hidet_status_t hidet_block_task(int32_t tiles_m, int32_t tiles_n, int32_t group, int32_t w, int32_t* tile_i,
                                int32_t* tile_j) {
  if (tiles_m <= 0 || tiles_n <= 0 || group <= 0 || w < 0 || !tile_i || !tile_j) return HIDET_ERR_INVALID_ARG;
  const long long tiles = (long long)tiles_m * tiles_n;
  if (w >= tiles || tiles > kIntMax) return HIDET_ERR_INVALID_ARG;
  GemmParams p;
  set_block_mapping(p, tiles_m, tiles_n, group < tiles_m ? group : tiles_m);  // (as a launch does)
  const tmap::Task t = grouped_tile(p, w);
  *tile_i = t.i;
  *tile_j = t.j;
  return HIDET_OK;
}

hidet_status_t hidet_host_div(int64_t divisor, int32_t n, int32_t* quotient) {
  if (divisor <= 0 || divisor > kIntMax || n < 0 || !quotient) return HIDET_ERR_INVALID_ARG;
  *quotient = make_fastdiv(divisor).div(n);
  return HIDET_OK;
}

const char* hidet_status_string(int32_t status) {
  switch (status) {
    case HIDET_OK: return "ok";
    case HIDET_ERR_INVALID_ARG: return "invalid argument";
    case HIDET_ERR_UNSUPPORTED: return "unsupported";
    case HIDET_ERR_ALIGNMENT: return "misaligned pointer";
    case HIDET_ERR_NO_CONFIG: return "no applicable tile configuration";
    case HIDET_ERR_LAUNCH: return "kernel launch failed";
    case HIDET_ERR_SCRATCH: return "partial sums exceed the static scratch array";
    default: return "unknown status";
  }
}

const char* hidet_version(void) { return "hidet-mi355x 0.1 (gfx950)"; }

int64_t hidet_kernel_launch_count(void) { return g_kernel_launches; }

}  // extern "C"

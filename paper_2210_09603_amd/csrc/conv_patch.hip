// 3x3 and 5x5 convolutions of unit stride, the output as large as the input, from a patch of the input in LDS.
//
// The img2col gather fetches every input value nine (25) times through the first-level cache, with a mask and about 45 vector
// instructions for each chunk of eight, and that bounds it, not the matrix cores (64 images of 256x14x14, 256 channels: 37.7
// us, 390 TFLOP/s).  Here a workgroup fetches its part of the input once for each 16 channels and multiplies it for every tap.
//
//   columns   The output columns run through a plane with one zero column behind every row and one zero row behind every
//             image (two of each for 5x5), n = (image * (H + 1) + row) * (W + 1) + column, so that filter tap (kh, kw) of
//             every column is the pixel (kh - 1) * (W + 1) + (kw - 1) further on: a zero where the filter leaves the image,
//             whichever side it leaves on (of the columns 1.15 times as many as outputs at 14x14, 1.07 at 28x28; the padding in
//             the gather's columns is 1.14).  Columns of zeros are computed and never stored.
//   patch     [2 x 8 channels][256 pixels][8] in LDS, two of them: the 128 columns of the tile and W + 2 pixels on either side.
//             A thread has two neighbouring pixels for the whole kernel, so their address and which of them are zeros are
//             worked out once.  The channels of a pixel lie together, so a fragment is one 16-byte read whatever the tap.
//   weights   As they lie in memory: 16 channels of a row are 144 values, of which a lane needs eight channels of all nine
//             taps, 144 consecutive bytes.  It reads them as nine 16-byte pieces and forms the nine fragments by 36 byte
//             permutations.  Rows are 19 chunks apart in LDS (an odd number: reads of consecutive rows meet in no bank).
//
// A stage is 16 channels, nine k steps of the 32x32x16 matrix instruction.  What bounds it is the rate at which a compute unit
// takes load instructions (timestamps: with those of a stage at its start, wavefronts wait 1000 to 1400 of its 3100 cycles to
// issue them, the 18 matrix instructions take 850), so they and the writes to LDS go between the taps, two stages ahead.  64
// images of 256x14x14, 256 channels: 32.5 us pixel by pixel and at the start of a stage, 27.7 us by pairs of pixels, 26.1 us
// between the taps.  (Four pixels a load: 26.3 us.)  45 us -> 30 us for 128x28x28, 46 -> 32 us for 512x7x7, 50 -> 37 us for
// 64x56x56, 64 images each; 99 -> 42 us for 68 images of 192x21x21.
// What is left has no single bound.  For a stage the LDS reads 27 KB of fragments for each of eight wavefronts, 907 cycles (244
// bytes a clock for these addresses), and a SIMD's 36 matrix instructions take 1152; without loads, deposits and stores a stage
// lasts 1970, as long as one after the other, and with them 3300 (27.4 us with all of them, 24.1 without the loads, 19.0 without
// any).  Of these the matrix cores work 35 %, the LDS 48 % (a fifth of it bank conflicts), the first-level cache 61 %; wavefronts
// spend 32 % at wait counts and barriers and 40 % waiting to issue.  (The barrier before the last filter row, with the fragments of
// the next stage read under it: 24.1 us; wave tiles of 64x64, which read a third less, one to a SIMD: 30.8 us.)
// 5x5: 25 taps take 100 registers of weights and 60 more for each stage on its way, so there is one wavefront to a SIMD (64 rows
// alone).  With one stage on its way instead of two the wavefront waited for the weights for as long as it computed: 20 of
// 256x14x14 50.7 us, 32.0 with two; 47 of 512x7x7 94 -> 63.5 us, 15 of 128x29x29 28 -> 21.
#include "epilogue.hpp"

namespace hidet {

// SETS_: stages on their way in registers.  (A single one has no use for a second: 15 of 16x10x10, 5x5, 394 channels: 7.3 us, 8.0.)
template <int BM, int KW, int SETS_ = 2>
struct PatchConv {
  static constexpr int BN = 128, IC_STEP = 16, PIXELS = 256, TAPS = KW * KW, PAD = KW / 2;
  static constexpr int WAVES_M = BM / 32, WAVES_N = 2, NT = WAVES_M * WAVES_N * 64;
  static constexpr int FN = BN / WAVES_N / 32;               // matrix-core tiles of a wavefront, 32 x 64
  static constexpr int CHUNKS = 2 * TAPS, PITCH = CHUNKS + 1;  // of a row of the weights: for one stage, and from row to row in LDS
  static constexpr int NL = (BM * CHUNKS + NT - 1) / NT;     // chunks of the weights that a thread loads for one stage
  static constexpr int A_BYTES = BM * PITCH * 16, P_BYTES = PIXELS * IC_STEP * 2;
  static constexpr int CHANNELS = PIXELS / 2 * IC_STEP / NT; // of the two pixels of the patch that a thread fetches
  static constexpr int SETS = SETS_;
  static constexpr int PER_SIMD = KW == 3 ? 2 : 1;           // wavefronts, which the LDS of a workgroup allows
  // after which taps of a stage the pixels and the weights of another one are requested
  static constexpr int PIECES = CHANNELS == 8 ? 4 : 1, FIRST_W = CHANNELS == 8 ? 4 : 2;
  static_assert(FIRST_W + NL <= TAPS, "a piece after each tap");
  static_assert(BM % 32 == 0 && (CHANNELS == 4 || CHANNELS == 8), "whole wavefronts and pieces of a pixel");
};

template <typename T, int BM, int KW, int SETS, class S = PatchConv<BM, KW, SETS>>
__global__ void __launch_bounds__(S::NT, S::PER_SIMD) conv_patch_kernel(const GemmParams p) {
  using Frag = typename FragT<T>::type;
  constexpr int BN = S::BN, NT = S::NT, FN = S::FN;
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * (S::A_BYTES + S::P_BYTES)];
  unsigned char* const patches = smem + 2 * S::A_BYTES;

  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const BlockCoords bc = block_coords<BM, BN>(p);
  const int wm0 = (wave / S::WAVES_N) * 32, wn0 = (wave % S::WAVES_N) * (FN * 32);
  const int W = p.g.W, H = p.g.H, HW = p.g.HW, pitch = W + S::PAD;

  // ---- this thread's pixels of the patch: two neighbours (the first of them an even one), S::CHANNELS channels
  const T* const x = reinterpret_cast<const T*>(p.B);
  const int reach = S::PAD * pitch + S::PAD;  // how far the first tap lies before a column
  const int border = (reach + 1) & ~1;       // pixels of the patch before the tile's first column
  const int pair = tid % (S::PIXELS / 2), ch0 = tid / (S::PIXELS / 2) * S::CHANNELS;
  unsigned xoff, keep0, keep1;
  int down;  // by how many bits the pair is to be shifted down
  {
    const int v = bc.n0 - border + 2 * pair;
    const int row = p.g.d_owp.div(v < 0 ? 0 : v), col = v - row * pitch;      // (d_owp: by W + PAD, d_oh: by H + PAD)
    const int img = p.g.d_oh.div(row), ih = row - img * (H + S::PAD);
    const bool real = v >= 0 && v < p.N;
    const bool in0 = real && col < W && ih < H;
    // the second one: in the same row, or the first of the next row, of the next image
    const bool wraps = col == pitch - 1, under = ih == H + S::PAD - 1;
    const int img1 = wraps && under ? img + 1 : img, ih1 = wraps ? (under ? 0 : ih + 1) : ih, col1 = wraps ? 0 : col + 1;
    const bool in1 = v >= 0 && v + 1 < p.N && col1 < W && ih1 < H;
    keep0 = in0 ? 0xffffffffu : 0u;
    keep1 = in1 ? 0xffffffffu : 0u;
    // where the second one lies, less one, is where the first does or a value that is not kept; v = 0 begins a pair, so
    // nothing lies before the tensor
    const unsigned at0 = ((unsigned)(img * p.g.IC + ch0) * (unsigned)H + (unsigned)ih) * (unsigned)W + (unsigned)col;
    const unsigned at1 = ((unsigned)(img1 * p.g.IC + ch0) * (unsigned)H + (unsigned)ih1) * (unsigned)W + (unsigned)col1;
    xoff = in0 ? at0 : in1 ? at1 - 1u : 0u;
    // the last pixel of the tensor would be followed by a value outside it (of its last channel): one value further down
    const bool last = in0 && !in1 && img == p.g.d_oh.div(p.g.d_owp.div(p.N - 1)) && ih == H - 1;
    down = last ? 16 : 0;
    if (last) xoff -= 1u;
  }

  // ---- this thread's chunks of the weights
  const T* const w = reinterpret_cast<const T*>(p.A) + (long long)bc.m0 * p.lda;
  unsigned woff[S::NL];
  int wat[S::NL];
#pragma unroll
  for (int q = 0; q < S::NL; ++q) {
    const int pos = q * NT + tid < BM * S::CHUNKS ? q * NT + tid : BM * S::CHUNKS - 1;  // (threads beyond the last chunk repeat it)
    const int row = pos / S::CHUNKS, c = pos % S::CHUNKS, left = p.M - bc.m0;
    woff[q] = (unsigned)(row < left ? row : left - 1) * (unsigned)p.lda + (unsigned)c * 8u;
    wat[q] = row * (S::PITCH * 16) + c * 16;
  }

  struct __attribute__((packed, aligned(2))) Pair {
    unsigned v;
  };
  struct Loads {  // a stage on its way
    unsigned px[S::CHANNELS];
    u32x4 wt[S::NL];
  };
  const int stages = p.g.IC / S::IC_STEP;
  // (stages beyond the last repeat it: the loads in flight are the same number whatever the stage)
  auto request_pixels = [&](Loads& l, int s, int piece) {
    const int at = s < stages ? s : stages - 1;
#pragma unroll
    for (int j = piece * S::CHANNELS / S::PIECES; j < (piece + 1) * S::CHANNELS / S::PIECES; ++j)
      l.px[j] = reinterpret_cast<const Pair*>(x + (long long)(at * S::IC_STEP + j) * HW + xoff)->v;
  };
  auto request_weights = [&](Loads& l, int s, int q) {
    l.wt[q] = *reinterpret_cast<const u32x4*>(w + (s < stages ? s : stages - 1) * (S::IC_STEP * S::TAPS) + woff[q]);
  };
  auto deposit_pixels = [&](Loads& l, int s) {
    unsigned v0[S::CHANNELS / 2], v1[S::CHANNELS / 2];
#pragma unroll
    for (int i = 0; i < S::CHANNELS / 2; ++i) {
      asm volatile("" : "+v"(l.px[2 * i]), "+v"(l.px[2 * i + 1]));  // (joined here, not as they arrive)
      const unsigned a = l.px[2 * i] >> down, b = l.px[2 * i + 1] >> down;
      v0[i] = __builtin_amdgcn_perm(b, a, 0x05040100u) & keep0;
      v1[i] = __builtin_amdgcn_perm(b, a, 0x07060302u) & keep1;
    }
    unsigned char* const at = patches + (s & 1) * S::P_BYTES + (ch0 / 8 * S::PIXELS + 2 * pair) * 16 + ch0 % 8 * 2;
    __builtin_memcpy(__builtin_assume_aligned(at, S::CHANNELS * 2), v0, S::CHANNELS * 2);
    __builtin_memcpy(__builtin_assume_aligned(at + 16, S::CHANNELS * 2), v1, S::CHANNELS * 2);
  };
  auto deposit_weights = [&](Loads& l, int s, int q) {
    *reinterpret_cast<u32x4*>(smem + (s & 1) * S::A_BYTES + wat[q]) = l.wt[q];
  };

  f32x16 acc[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;

  const int a_at = (wm0 + lane % 32) * (S::PITCH * 16) + (lane / 32) * (S::TAPS * 16);
  const int b_at = ((lane / 32) * S::PIXELS + border - reach + wn0 + lane % 32) * 16;
  // Stage s is multiplied; meanwhile, a piece after each tap, stage s + 1 (in `l`) goes to LDS and another one is requested in
  // its place, two stages ahead of its use.
  auto step = [&](int s, Loads& l) {
    const unsigned char* a = smem + (s & 1) * S::A_BYTES + a_at;
    const unsigned char* b = patches + (s & 1) * S::P_BYTES + b_at;
    // fragments of the input for the taps of a filter row, read a row ahead
    Frag fb[2][KW][FN];
    auto read_row = [&](int kh) {
#pragma unroll
      for (int kw = 0; kw < KW; ++kw)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          fb[kh & 1][kw][j] = __builtin_bit_cast(Frag, *reinterpret_cast<const u32x4*>(b + (kh * pitch + kw + j * 32) * 16));
    };
    unsigned raw[4 * S::TAPS];
#pragma unroll
    for (int c = 0; c < S::TAPS; ++c) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(a + c * 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) raw[4 * c + i] = v[i];
    }
    read_row(0);
#pragma unroll
    for (int kh = 0; kh < KW; ++kh) {
      if (kh + 1 < KW) read_row(kh + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kw = 0; kw < KW; ++kw) {
        const int t = kh * KW + kw;
        u32x4 f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // channels 2i, 2i + 1 of tap t
          const int e0 = 2 * S::TAPS * i + t, e1 = e0 + S::TAPS;
          f[i] = __builtin_amdgcn_perm(raw[e1 / 2], raw[e0 / 2], e0 % 2 == 0 ? 0x07060100u : 0x05040302u);
        }
        const Frag fa = __builtin_bit_cast(Frag, f);
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[j] = mfma_op(fa, fb[kh & 1][kw][j], acc[j]);
        if (t == 0) deposit_pixels(l, s + 1);
        if (t >= 1 && t <= S::PIECES) request_pixels(l, s + 1 + S::SETS, t - 1);
        if (t >= S::FIRST_W && t - S::FIRST_W < S::NL) {
          deposit_weights(l, s + 1, t - S::FIRST_W);
          request_weights(l, s + 1 + S::SETS, t - S::FIRST_W);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
  };
  Loads l[S::SETS];
  auto request = [&](Loads& r, int s) {
#pragma unroll
    for (int i = 0; i < S::PIECES; ++i) request_pixels(r, s, i);
#pragma unroll
    for (int q = 0; q < S::NL; ++q) request_weights(r, s, q);
  };
#pragma unroll
  for (int s = 0; s < S::SETS; ++s) request(l[s], s);
  deposit_pixels(l[0], 0);
#pragma unroll
  for (int q = 0; q < S::NL; ++q) deposit_weights(l[0], 0, q);
  request(l[0], S::SETS);
  __syncthreads();
  int s = 0;
  for (; s + 1 < stages; s += 2) {  // (two by two and without a branch: registers on their way must not be moved)
    step(s, l[S::SETS - 1]);
    step(s + 1, l[0]);
  }
  if (s < stages) step(s, l[S::SETS - 1]);

  // ---- epilogue, from the accumulators: a lane holds one column, 16 rows; the two halves of a wavefront store 32 consecutive
  // pixels of one row each.  (Through LDS, in groups of four pixels gathered from between the zero columns and stored by 8 bytes:
  // 64 images of 256x14x14 32.0 us instead of 26 to 28, 64x56x56 47.7 us instead of 38.)
  const T* const bias = reinterpret_cast<const T*>(p.bias);
  const T* const R = reinterpret_cast<const T*>(p.residual);
  T* const C = reinterpret_cast<T*>(p.C);
  const int m_lane = bc.m0 + wm0 + (lane / 32) * 4;  // row of accumulator r: m_lane + (r / 4) * 8 + r % 4
  float badd[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) badd[r] = 0.0f;
  if (p.bias_axis == 2) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m_lane + (r / 4) * 8 + r % 4;
      badd[r] = to_f32(bias[m < p.M ? m : 0]);
    }
  }
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int n = bc.n0 + wn0 + j * 32 + lane % 32;
    const int row = p.g.d_owp.div(n), col = n - row * pitch;
    const int img = p.g.d_oh.div(row), oh = row - img * (H + S::PAD);
    const bool output = n < p.N && col < W && oh < H;
    const long long at = output ? (long long)img * p.out_outer + oh * W + col : 0;
    float v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = p.alpha * acc[j][r] + badd[r];
    if (R != nullptr) {
      T res[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {  // (requested together: clamped, not predicated)
        const int m = m_lane + (r / 4) * 8 + r % 4;
        res[r] = R[at + (long long)(m < p.M ? m : p.M - 1) * HW];
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] += to_f32(res[r]);
    }
    if (!output) continue;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m_lane + (r / 4) * 8 + r % 4;
      if (p.relu) v[r] = v[r] < 0.0f ? 0.0f : v[r];
      if (m < p.M) C[at + (long long)m * HW] = from_f32<T>(v[r]);
    }
  }
}

template <typename T, int BM, int KW, int SETS = 2>
hipError_t launch_tiles(const GemmParams& p, hipStream_t stream) {
  hipLaunchKernelGGL((conv_patch_kernel<T, BM, KW, SETS>), dim3((unsigned)p.total_blocks), dim3(PatchConv<BM, KW>::NT), 0, stream, p);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_type(const GemmParams& p, int bm, hipStream_t stream) {
  if (p.g.KW == 5) return p.g.IC <= 16 ? launch_tiles<T, 64, 5, 1>(p, stream) : launch_tiles<T, 64, 5>(p, stream);
  return bm == 64 ? launch_tiles<T, 64, 3>(p, stream) : launch_tiles<T, 128, 3>(p, stream);
}

hipError_t launch_conv_patch_f16(const GemmParams& p, int bm, hipStream_t stream) { return launch_type<f16>(p, bm, stream); }
hipError_t launch_conv_patch_bf16(const GemmParams& p, int bm, hipStream_t stream) { return launch_type<bf16>(p, bm, stream); }

}  // namespace hidet

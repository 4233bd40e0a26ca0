// Table of compiled kernels: [tile configuration][input type][variant] -> launcher.
#pragma once

#include <hip/hip_runtime.h>

#include "gemm_kernel.hpp"
#include "wave_kernel.hpp"

namespace hidet {

using LaunchFn = hipError_t (*)(const GemmParams&, hipStream_t);

constexpr int kMaxConfigs = 64;
constexpr int kNumTypes = 3;     // index = hidet_dtype_t of the inputs: 0 f32, 1 f16, 2 bf16 (output has the same type)
constexpr int kNumVariants = 23; // GEMM: transA*4 + transB*2 + mode (0 vector loads, 1 element loads); conv: 8 + mode;
                                 // +10: the same operand forms writing raw fp32 partial sums to a plain [M][N]
                                 // workspace (first pass of the parallel reduction on K);
                                 // 20, 21: convolution with repacked (tap-major) weights, and its partial-sum form;
                                 // 22: 1x1 convolution whose columns run through all images (ring schedule)

struct ConfigRow {
  int index, bm, bn, bk, waves_m, waves_n, mfma, trans_a, sched, is_f32;
};

struct Registry {
  LaunchFn fn[kMaxConfigs][kNumTypes][kNumVariants];
};

inline int gemm_variant(int transA, int transB, int elem_mode) { return (transA ? 4 : 0) + (transB ? 2 : 0) + (elem_mode ? 1 : 0); }
inline int conv_variant(int elem_mode) { return 8 + (elem_mode ? 1 : 0); }
constexpr int kPartialVariants = 10;  // offset of the K-parallel partial-sum kernels
constexpr int kPointwiseVariant = 22;
constexpr int kConvTapVariant = 20;   // convolution over the tap-major K order (repacked weights); +1: partial sums

// Largest leading dimension for vector loads: in-tile element offsets (row * ld + col, row < 512) stay below 2^31.
constexpr long long kMaxVecLd = 4LL << 20;

// Whether direct loads on element-aligned operands stay where they belong.  Their offsets inside a tile are unsigned 32-bit
// byte offsets (Operand::init_direct), and the 16 bytes that begin in the last columns of an M/N-contiguous operand must not
// reach past the row that follows.  What remains goes through registers on the same tile.
constexpr bool direct_offsets_fit(long long rows, long long ld) { return ld <= (1LL << 31) / rows; }  // (of 16-bit elements)
template <class Cfg>
bool direct_loads_fit(const GemmParams& p) {
  static_assert(Cfg::MODE_A == LD_ELEM && Cfg::MODE_B == LD_ELEM, "rows of aligned operands are whole chunks, kMaxVecLd apart at most");
  return direct_offsets_fit(Cfg::LA == L_KC ? Cfg::BM : Cfg::BK, p.lda) && direct_offsets_fit(Cfg::LB == L_KC ? Cfg::BN : Cfg::BK, p.ldb) &&
         (Cfg::LA == L_KC || p.lda >= Cfg::VEC) && (Cfg::LB == L_KC || p.ldb >= Cfg::VEC);
}

// Tiles of products that can be as short as their launch (see PlainParams).
template <class Cfg>
constexpr bool kSmallPlain = Cfg::MAPPER == MAP_PLAIN && std::is_same<typename Cfg::T, typename Cfg::TO>::value &&
                             !Cfg::GATHER_B && Cfg::MODE_B != LD_IMAGES && Cfg::BM * Cfg::BN <= 64 * 64;

template <class Cfg>
constexpr bool kWavesF32 = Cfg::IS_F32 && Cfg::SCHED == SCHED_KSPLIT && Cfg::MAPPER == MAP_PLAIN && !Cfg::GATHER_B;

// (see gemm_kernel_waves_direct for where it is taken)
template <class Cfg>
constexpr bool kWavesDirect = Cfg::BM == 16 && Cfg::BN <= 32 && Cfg::LA == L_KC && Cfg::LB == L_MC;

template <class Cfg>
hipError_t launch_kernel(const GemmParams& p, hipStream_t stream) {
  const dim3 grid((unsigned)p.total_blocks);
  constexpr bool ELEM = Cfg::MODE_A == LD_ELEM, RING = Cfg::SCHED == SCHED_PINGPONG, WAVES = WaveStream<Cfg>::BUILT;
  static_assert(!(RING || WAVES) || direct_offsets_fit(Cfg::BM > Cfg::BN ? Cfg::BM : Cfg::BN, kMaxVecLd), "rows of a tile");
  static_assert(!(RING || WAVES) || direct_offsets_fit(Cfg::BK, kMaxVecLd), "rows of a tile");
  if constexpr (kWavesF32<Cfg>) {  // (at any alignment)
    constexpr int BM = Cfg::BM, BN = Cfg::BN;
    if (PlainParams c; plain_params(p, c))
      hipLaunchKernelGGL((gemm_kernel_waves_f32<BM, BN, Cfg::LA, Cfg::LB, PlainParams>), grid, dim3(WaveStreamF32<BM, BN>::NT), 0, stream, c);
    else
      hipLaunchKernelGGL((gemm_kernel_waves_f32<BM, BN, Cfg::LA, Cfg::LB, GemmParams>), grid, dim3(WaveStreamF32<BM, BN>::NT), 0, stream, p);
  } else if constexpr (RING) {
    // the element-mode variant of a ring tile also serves what the direct loads cannot do (input prologue, head-split
    // output map, rows too far apart or too short), with its stages staged through registers
    if constexpr (ELEM) {
      if (p.out_map != 0 || p.relu_a != 0 || p.relu_b != 0 || !direct_loads_fit<Cfg>(p)) {
        hipLaunchKernelGGL(gemm_kernel_pingpong_regs<Cfg>, grid, dim3(Cfg::NT), 0, stream, p);
        return hipGetLastError();
      }
    }
    // a K range of at most two stages never reuses a ring slot: the two-slot form leaves LDS for a second workgroup
    const int k_len = p.k_slices > 1 ? p.k_slice_len : p.K;
    if (k_len <= 2 * Cfg::BK)
      hipLaunchKernelGGL((gemm_kernel_pingpong<Cfg, 2>), grid, dim3(Cfg::NT), 0, stream, p);
    else
      hipLaunchKernelGGL((gemm_kernel_pingpong<Cfg, 4>), grid, dim3(Cfg::NT), 0, stream, p);
  } else if constexpr (WAVES) {
    if constexpr (ELEM) {
      if constexpr (kWavesDirect<Cfg>) {
        using T = typename Cfg::T;
        using TO = typename Cfg::TO;
        using S = WaveDirect<Cfg::BM, Cfg::BN>;
        const bool fit = direct_loads_fit<Cfg>(p);
        const bool even = (((unsigned long long)p.A / 2 | (unsigned long long)p.lda | (unsigned long long)p.strideA) & 1) == 0;
        const bool few_k = (p.k_slices > 1 ? p.k_slice_len : p.K) <= S::MAX_K;
        const bool narrow = (p.k_slices > 1 ? p.k_slice_len : p.K) > 768LL * p.N - 512;
        if (p.N >= 2 && (even ? !fit || few_k : !fit && few_k && !narrow)) {
          if (PlainParams c; plain_params(p, c))
            hipLaunchKernelGGL((gemm_kernel_waves_direct<T, TO, Cfg::BM, Cfg::BN, PlainParams>), grid, dim3(S::NT), 0, stream, c);
          else
            hipLaunchKernelGGL((gemm_kernel_waves_direct<T, TO, Cfg::BM, Cfg::BN, GemmParams>), grid, dim3(S::NT), 0, stream, p);
          return hipGetLastError();
        }
      }
      if (!direct_loads_fit<Cfg>(p)) {
        hipLaunchKernelGGL((gemm_kernel<Cfg, GemmParams>), grid, dim3(Cfg::NT), 0, stream, p);
        return hipGetLastError();
      }
    }
    if constexpr (kSmallPlain<Cfg>) {
      if (PlainParams c; plain_params(p, c)) {
        hipLaunchKernelGGL((gemm_kernel_waves<Cfg, PlainParams>), grid, dim3(WaveStream<Cfg>::NT), 0, stream, c);
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((gemm_kernel_waves<Cfg, GemmParams>), grid, dim3(WaveStream<Cfg>::NT), 0, stream, p);
  } else {
    if constexpr (kSmallPlain<Cfg>) {
      if (PlainParams c; plain_params(p, c)) {
        hipLaunchKernelGGL((gemm_kernel<Cfg, PlainParams>), grid, dim3(Cfg::NT), 0, stream, c);
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((gemm_kernel<Cfg, GemmParams>), grid, dim3(Cfg::NT), 0, stream, p);
  }
  return hipGetLastError();
}

// Fills the launchers of one (configuration, input type) pair.
template <typename T, int BM, int BN, int BK, int WM, int WN, int MI, int TRANS_A, int SCHED>
void register_config(Registry& r, int index, int type_index) {
  LaunchFn* v = r.fn[index][type_index];
  // the operand forms that the ring schedule does not cover run the general kernel on the same tile
  constexpr int GS = (SCHED == SCHED_PINGPONG) ? SCHED_SIMPLE : SCHED;
  // row-major A: KC;  row-major B: MC;  transposed B: KC;  transposed A: MC
  v[gemm_variant(0, 0, 0)] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_KC, L_MC, LD_VEC, LD_VEC, MAP_PLAIN, SCHED>>;
  v[gemm_variant(0, 0, 1)] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_KC, L_MC, LD_ELEM, LD_ELEM, MAP_PLAIN, SCHED>>;
  v[gemm_variant(0, 1, 0)] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_KC, L_KC, LD_VEC, LD_VEC, MAP_PLAIN, SCHED>>;
  v[gemm_variant(0, 1, 1)] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_KC, L_KC, LD_ELEM, LD_ELEM, MAP_PLAIN, SCHED>>;
  if constexpr (TRANS_A != 0) {
    v[gemm_variant(1, 0, 0)] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_MC, L_MC, LD_VEC, LD_VEC, MAP_PLAIN, SCHED>>;
    v[gemm_variant(1, 0, 1)] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_MC, L_MC, LD_ELEM, LD_ELEM, MAP_PLAIN, SCHED>>;
    v[gemm_variant(1, 1, 0)] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_MC, L_KC, LD_VEC, LD_VEC, MAP_PLAIN, SCHED>>;
    v[gemm_variant(1, 1, 1)] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_MC, L_KC, LD_ELEM, LD_ELEM, MAP_PLAIN, SCHED>>;
  }
  // convolution: weights are a row-major OC x (IC*KH*KW) matrix, B is the img2col gather, C is NCHW
  v[conv_variant(0)] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_KC, L_MC, LD_VEC, LD_IM2COL, MAP_NCHW, GS>>;
  v[conv_variant(1)] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_KC, L_MC, LD_ELEM, LD_IM2COL, MAP_NCHW, GS>>;
  v[kConvTapVariant] = launch_kernel<GemmConfig<T, T, BM, BN, BK, WM, WN, MI, L_KC, L_MC, LD_VEC, LD_IM2COL_TAP, MAP_NCHW, GS>>;
  // 1x1 convolution over all images: stages of 32, whose ring takes 64 KB, so that two workgroups share a compute unit and the
  // output write of one overlaps the loads and the products of the other (64 images of 512x7x7, 2048 channels, with residual:
  // 18.4 us, 23.8 us with stages of 64; 256x128 tiles of stages of 32, one to a compute unit: 20.2 us; 256x256: 31.4 us)
  if constexpr (SCHED == SCHED_PINGPONG && BM == 128 && BN == 128)
    v[kPointwiseVariant] = launch_kernel<GemmConfig<T, T, BM, BN, 32, WM, WN, MI, L_KC, L_MC, LD_VEC, LD_IMAGES, MAP_NCHW, SCHED>>;
  // K-parallel partial sums (fp32 out, plain map): built for the small and medium tiles, which are the ones a
  // problem with few output tiles and a long K wants, and for the ring-schedule tiles (medium-sized problems whose
  // tiles do not fill the device)
  if constexpr (BM * BN <= 128 * 128 || SCHED == SCHED_PINGPONG) {
    LaunchFn* w = v + kPartialVariants;
    w[gemm_variant(0, 0, 0)] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_KC, L_MC, LD_VEC, LD_VEC, MAP_PLAIN, SCHED>>;
    w[gemm_variant(0, 0, 1)] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_KC, L_MC, LD_ELEM, LD_ELEM, MAP_PLAIN, SCHED>>;
    w[gemm_variant(0, 1, 0)] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_KC, L_KC, LD_VEC, LD_VEC, MAP_PLAIN, SCHED>>;
    w[gemm_variant(0, 1, 1)] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_KC, L_KC, LD_ELEM, LD_ELEM, MAP_PLAIN, SCHED>>;
    if constexpr (TRANS_A != 0) {
      w[gemm_variant(1, 0, 0)] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_MC, L_MC, LD_VEC, LD_VEC, MAP_PLAIN, SCHED>>;
      w[gemm_variant(1, 0, 1)] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_MC, L_MC, LD_ELEM, LD_ELEM, MAP_PLAIN, SCHED>>;
      w[gemm_variant(1, 1, 0)] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_MC, L_KC, LD_VEC, LD_VEC, MAP_PLAIN, SCHED>>;
      w[gemm_variant(1, 1, 1)] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_MC, L_KC, LD_ELEM, LD_ELEM, MAP_PLAIN, SCHED>>;
    }
    w[conv_variant(0)] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_KC, L_MC, LD_VEC, LD_IM2COL, MAP_PLAIN, GS>>;
    w[conv_variant(1)] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_KC, L_MC, LD_ELEM, LD_IM2COL, MAP_PLAIN, GS>>;
    v[kConvTapVariant + 1] = launch_kernel<GemmConfig<T, float, BM, BN, BK, WM, WN, MI, L_KC, L_MC, LD_VEC, LD_IM2COL_TAP, MAP_PLAIN, GS>>;
  }
}

// Second pass of the parallel reduction on K: [output type index][0 plain map, 1 NCHW map].
template <typename TO, int MAPPER>
hipError_t launch_reduce(const GemmParams& p, int batch, hipStream_t stream) {
  const long long groups = (long long)p.M * ((p.N + 3) / 4);
  hipLaunchKernelGGL((splitk_reduce_kernel<TO, MAPPER>), dim3((unsigned)((groups + 255) / 256), (unsigned)batch), dim3(256), 0,
                     stream, p);
  return hipGetLastError();
}

}  // namespace hidet

// Reduction schedule template (the second of the two templates the Hidet paper schedules by hand:
// reductions such as a sum along one axis; end of Section 5) and the row softmax built from it.
//
// Both operations are memory bound: a row is read once and (softmax) written once.  The schedule is a
// task mapping in the sense of Section 5.1 over the [rows, 16-byte chunks] grid of the input; as long as
// a row fits, it sits in registers between the passes over it (max, exp and sum, write):
//
//   wavefront    workgroup = 4 wavefronts; wavefront = spatial(64 / L, L) over (rows, chunks) composed
//                with repeat(1, R): L lanes share one row, lane c of the group owns chunks c, c + L, ...;
//                lanes combine with xor butterflies (L is a power of two).
//   workgroup    workgroup = spatial(1, NT) over the chunks of one row composed with repeat(1, R): rows too
//                long for one wavefront's registers, and medium rows of which there are too few to give
//                every compute unit several wavefronts.  The wavefronts' results meet in LDS.
//   streamed     rows of more than 16384 chunks, and reductions of many rows of more than 1024 whole (8192
//                ragged) chunks: one workgroup per row, a running (max, sum) pair per thread, merged through
//                LDS; softmax re-reads the row (from L2 when it fits).
//
// Chunks are accessed at element alignment (16-byte loads and stores take any element-aligned address
// here), so rows of any length and leading dimension run the same way.  The last chunk of a row whose
// length is no multiple of a chunk is loaded from the 16 bytes that end the row; its elements that
// belong to the chunk before are masked out.
//
// Arithmetic is fp32 whatever the storage type.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/hidet_mi355x.h"
#include "gemm_kernel.hpp"

using namespace hidet;

namespace {

struct RowParams {
  const void* x;
  void* y;
  long long ldx, ldy;
  long long rows;
  int cols;
  int op;       // reduce: hidet_reduce_op_t
  int out_f32;  // reduce: y is fp32 whatever T is
  int shift;    // softmax: rows of y are not all 16-byte aligned (see row_shift)
};

constexpr float kNegInf = -__builtin_huge_valf();

template <typename T>
struct Chunk {
  static constexpr int VEC = 16 / (int)sizeof(T);
  struct __attribute__((packed, aligned(sizeof(T)))) Raw {  // 16 bytes at element alignment
    u32x4 v;
  };
  typedef u32x4 Streamed __attribute__((aligned(2)));  // (the same, for a store with a hint)
};

// The 16 bytes that hold the elements of chunk [col0, col0 + VEC) of a row: the chunk itself, or, where it would stick
// out of the row at either end, the first or last 16 bytes of the row.  Always a valid address, so that the loads of all
// of a thread's chunks can be in flight together.  (Rows shorter than one chunk: load_short.)
template <typename T>
__device__ __forceinline__ int chunk_pos(int col0, int cols) {
  const int last = cols - Chunk<T>::VEC;
  const int pos = col0 < last ? col0 : last;
  return pos > 0 ? pos : 0;
}
template <typename T>
__device__ __forceinline__ u32x4 load_raw(const T* row, int col0, int cols) {
  return reinterpret_cast<const typename Chunk<T>::Raw*>(row + chunk_pos<T>(col0, cols))->v;
}

// Elements [lo, hi) of what load_raw returned belong to chunk [col0, col0 + VEC).
template <typename T>
__device__ __forceinline__ void chunk_range(int col0, int cols, int& lo, int& hi) {
  const int pos = chunk_pos<T>(col0, cols), end = col0 + Chunk<T>::VEC;
  lo = (col0 > 0 ? col0 : 0) - pos;
  hi = (end < cols ? end : cols) - pos;
}

template <typename T>
__device__ __forceinline__ void widen_chunk(u32x4 raw, float* v) {
  constexpr int VEC = Chunk<T>::VEC;
  T t[VEC];
  __builtin_memcpy(t, &raw, 16);
#pragma unroll
  for (int e = 0; e < VEC; ++e) v[e] = to_f32(t[e]);
}

// RAGGED: rows that are no whole number of chunks (or lie on a shifted grid); otherwise a chunk is inside or outside.
// `whole`: the caller knows that no lane's chunk sticks out (uniform: it costs no vector instructions).
template <typename T, bool RAGGED>
__device__ __forceinline__ void widen_masked(u32x4 raw, int col0, int cols, bool whole, float fill, float* v) {
  widen_chunk<T>(raw, v);
  if (whole) return;
  if constexpr (RAGGED) {
    int lo, hi;
    chunk_range<T>(col0, cols, lo, hi);
#pragma unroll
    for (int e = 0; e < Chunk<T>::VEC; ++e) v[e] = (e >= lo && e < hi) ? v[e] : fill;
  } else {
    const bool in = col0 < cols;
#pragma unroll
    for (int e = 0; e < Chunk<T>::VEC; ++e) v[e] = in ? v[e] : fill;
  }
}

// A row shorter than one chunk, element by element and by its first lane alone: with all lanes taking part, a sum over
// 700000 rows of one fp16 element took 12.2 us, 8.0 us this way (softmax 20.5 and 14.0 us).
template <typename T>
__device__ __forceinline__ void load_short(const T* row, int sub, int cols, float fill, float* v) {
#pragma unroll
  for (int e = 0; e < Chunk<T>::VEC; ++e) v[e] = fill;
  if (sub == 0 && cols > 0) {  // (cols == 0: nothing may be read)
#pragma unroll
    for (int e = 0; e < Chunk<T>::VEC; ++e) {
      const bool in = e < cols;
      const T t = row[in ? e : 0];
      v[e] = in ? to_f32(t) : fill;
    }
  }
}
template <typename T>
__device__ __forceinline__ void store_short(T* row, int cols, const float* v) {
#pragma unroll
  for (int e = 0; e < Chunk<T>::VEC; ++e)
    if (e < cols) row[e] = from_f32<T>(v[e]);
}

// (a chunk that lies wholly outside the row stores nothing)
template <typename T, bool RAGGED, bool STREAM>
__device__ __forceinline__ void store_chunk(T* row, int col0, int cols, const float* v) {
  constexpr int VEC = Chunk<T>::VEC;
  T t[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) t[e] = from_f32<T>(v[e]);
  if (col0 >= 0 && col0 + VEC <= cols) {
    typename Chunk<T>::Raw raw;
    __builtin_memcpy(&raw.v, t, 16);
    if constexpr (STREAM)
      __builtin_nontemporal_store(raw.v, reinterpret_cast<typename Chunk<T>::Streamed*>(row + col0));
    else
      *reinterpret_cast<typename Chunk<T>::Raw*>(row + col0) = raw;
  } else if constexpr (RAGGED) {
    int lo, hi;
    chunk_range<T>(col0, cols, lo, hi);
    T* dst = row + chunk_pos<T>(col0, cols);
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      if (e >= lo && e < hi) dst[e] = t[e];
  }
}

// Chunks of a very long softmax row are laid on the 16-byte grid of the output row: the first one then begins `shift`
// elements before the row.  Loads do not mind where a chunk lies, stores do (1024 x 50257 bf16: 53.4 us with chunks on
// the row's own grid, 47.8 us with aligned stores), but both ends of a row are then stored element by element, which on
// shorter rows costs as much or more (4096 x 8201: 33 us either way; 1000 x 4095: 6.5 -> 9.1 us).
template <typename T>
__device__ __forceinline__ int row_shift(const RowParams& p, const T* yr) {
  return p.shift ? (int)((reinterpret_cast<uintptr_t>(yr) / sizeof(T)) % Chunk<T>::VEC) : 0;
}

// Butterflies over groups of 1, 2, 4, ... lanes.  Every group holds one value by the time it meets its neighbour, so the
// neighbour may be mirrored (lane 7 - i or 15 - i for i ^ 4 or i ^ 8) and its value comes with the operand of the next
// instruction; a read of another lane through the LDS crossbar instead is a round trip for each of the six steps.
template <int CTRL>
__device__ __forceinline__ float from_lane(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int O>  // a and b: the values of the two groups of O lanes that meet
__device__ __forceinline__ void meet(float v, float& a, float& b) {
  if constexpr (O <= 8) {
    a = v;
    b = from_lane<O == 1 ? 0xB1 : O == 2 ? 0x4E : O == 4 ? 0x141 : 0x140>(v);  // quad_perm x2, row_half_mirror, row_mirror
  } else {
    const unsigned u = __builtin_bit_cast(unsigned, v);
    if constexpr (O == 16) {
      const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
      a = __builtin_bit_cast(float, (unsigned)r[0]);
      b = __builtin_bit_cast(float, (unsigned)r[1]);
    } else {
      const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
      a = __builtin_bit_cast(float, (unsigned)r[0]);
      b = __builtin_bit_cast(float, (unsigned)r[1]);
    }
  }
}
template <int L, bool MAX, bool CROSSBAR = false>
__device__ __forceinline__ float over_lanes(float v) {
  if constexpr (CROSSBAR) {  // (see spreads_rows; lanes meet in the same order, so the sum has the same bits)
#pragma unroll
    for (int o = 1; o < L; o <<= 1) {
      const float w = __shfl_xor(v, o, 64);
      v = MAX ? fmaxf(v, w) : v + w;
    }
    return v;
  }
  float a, b;
  auto step = [&] { v = MAX ? fmaxf(a, b) : a + b; };
  if constexpr (L >= 2) { meet<1>(v, a, b); step(); }
  if constexpr (L >= 4) { meet<2>(v, a, b); step(); }
  if constexpr (L >= 8) { meet<4>(v, a, b); step(); }
  if constexpr (L >= 16) { meet<8>(v, a, b); step(); }
  if constexpr (L >= 32) { meet<16>(v, a, b); step(); }
  if constexpr (L >= 64) { meet<32>(v, a, b); step(); }
  return v;
}
template <int L, bool CROSSBAR = false>
__device__ __forceinline__ float group_max(float v) {
  return over_lanes<L, true, CROSSBAR>(v);
}
template <int L, bool CROSSBAR = false>
__device__ __forceinline__ float group_sum(float v) {
  return over_lanes<L, false, CROSSBAR>(v);
}

__device__ __forceinline__ void write_scalar(const RowParams& p, long long row, float v, int dtype_tag) {
  if (p.out_f32)
    reinterpret_cast<float*>(p.y)[row] = v;
  else if (dtype_tag == 1)
    reinterpret_cast<f16*>(p.y)[row] = from_f32<f16>(v);
  else if (dtype_tag == 2)
    reinterpret_cast<bf16*>(p.y)[row] = from_f32<bf16>(v);
  else
    reinterpret_cast<float*>(p.y)[row] = v;
}

template <typename T>
struct Tag {
  static constexpr int value = sizeof(T) == 4 ? 0 : (std::is_same<T, f16>::value ? 1 : 2);
};

// ---- the row lives in the registers of L lanes of a wavefront ----------------------------------------
// SHAPE: WHOLE chunks, RAGGED rows of at least one chunk, SHORT ones of less.
enum RowShape { WHOLE, RAGGED_END, SHORT };
template <typename T, int L, int R, RowShape SHAPE, bool SOFTMAX, bool STREAM, bool CROSSBAR>
__global__ void __launch_bounds__(256) rows_in_registers_kernel(const RowParams p) {
  constexpr int VEC = Chunk<T>::VEC;
  constexpr bool RAGGED = SHAPE != WHOLE;
  constexpr int G = 64 / L;  // rows per wavefront
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  const int sub = lane % L;
  const bool is_max = SOFTMAX || p.op == HIDET_REDUCE_MAX;
  const float fill = is_max ? kNegInf : 0.0f;
  const long long stride = (long long)gridDim.x * 4 * G;
  for (long long row = ((long long)blockIdx.x * 4 + wave) * G + lane / L; row < p.rows; row += stride) {
    const T* xr = reinterpret_cast<const T*>(p.x) + row * p.ldx;
    float v[R][VEC];
    if constexpr (SHAPE == SHORT) {
      load_short<T>(xr, sub, p.cols, fill, v[0]);
    } else {
      u32x4 raw[R];
#pragma unroll
      for (int r = 0; r < R; ++r) raw[r] = load_raw<T>(xr, (r * L + sub) * VEC, p.cols);
#pragma unroll
      for (int r = 0; r < R; ++r)
        // (one whole chunk each: masking costs less than finding out that it need not be masked, 3.9 against 4.1 us for
        // a sum of 100000 x 64 fp32)
        widen_masked<T, RAGGED>(raw[r], (r * L + sub) * VEC, p.cols, (RAGGED || R > 1) && (r + 1) * L * VEC <= p.cols, fill, v[r]);
    }
    float m = fill;
    if (is_max) {
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int e = 0; e < VEC; ++e) m = fmaxf(m, v[r][e]);
      m = group_max<L, CROSSBAR>(m);
    }
    if constexpr (SOFTMAX) {
      float s = 0.0f;
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          v[r][e] = __expf(v[r][e] - m);  // padding: exp(-inf) = 0
          s += v[r][e];
        }
      s = group_sum<L, CROSSBAR>(s);
      const float inv = 1.0f / s;
      T* yr = reinterpret_cast<T*>(p.y) + row * p.ldy;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int col0 = (r * L + sub) * VEC;
        if (col0 < p.cols) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) v[r][e] *= inv;
          if constexpr (SHAPE == SHORT)
            store_short<T>(yr, p.cols, v[r]);
          else
            store_chunk<T, RAGGED, STREAM>(yr, col0, p.cols, v[r]);
        }
      }
    } else {
      float out = m;
      if (!is_max) {
        float s = 0.0f;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int e = 0; e < VEC; ++e) s += v[r][e];
        s = group_sum<L, CROSSBAR>(s);
        out = p.op == HIDET_REDUCE_MEAN ? s / (float)p.cols : s;
      }
      if (sub == 0) write_scalar(p, row, out, Tag<T>::value);
    }
  }
}

// ---- the row lives in the registers of a workgroup ---------------------------------------------------------
// Every thread holds R chunks as they were loaded, four registers each (with the widened values kept instead, half as many
// bytes would be in flight per register).  The row is read once.

// The wavefronts' results, combined in a tree: one after another, every addition would round at the size of the whole
// (sums of 700 rows of 9001 fp32 differ from 64 bits by 4.7e-8 in the norm, by 6.8e-8 one after another).
template <int NW, bool MAX>
__device__ __forceinline__ float across_wavefronts(float* red, int lane, int wave, float x) {
  if (lane == 0) red[wave] = x;
  __syncthreads();
  return over_lanes<NW, MAX>(red[lane % NW]);
}

template <typename T, int NT, int R, bool RAGGED>
__global__ void __launch_bounds__(NT, R <= 8 ? 8 : 4) reduce_in_workgroup_kernel(const RowParams p) {
  constexpr int VEC = Chunk<T>::VEC, NW = NT / 64;
  __shared__ float red[NW];
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const bool is_max = p.op == HIDET_REDUCE_MAX;
  const float fill = is_max ? kNegInf : 0.0f;
  const long long row = blockIdx.x;
  const T* xr = reinterpret_cast<const T*>(p.x) + row * p.ldx;
  auto col_of = [&](int r) { return (r * NT + tid) * VEC; };
  auto needed = [&](int r) { return r * NT * VEC < p.cols; };  // (uniform)
  u32x4 raw[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    raw[r] = u32x4{0u, 0u, 0u, 0u};
    if (needed(r)) raw[r] = load_raw<T>(xr, col_of(r), p.cols);
  }
  float m = fill, s = 0.0f;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (needed(r)) {
      float v[VEC];
      widen_masked<T, RAGGED>(raw[r], col_of(r), p.cols, (r + 1) * NT * VEC <= p.cols, fill, v);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        if (is_max)
          m = fmaxf(m, v[e]);
        else
          s += v[e];
      }
    }
  }
  float out;
  if (is_max) {
    out = across_wavefronts<NW, true>(red, lane, wave, group_max<64>(m));
  } else {
    s = across_wavefronts<NW, false>(red, lane, wave, group_sum<64>(s));
    out = p.op == HIDET_REDUCE_MEAN ? s / (float)p.cols : s;
  }
  if (tid == 0) write_scalar(p, row, out, Tag<T>::value);
}

// The largest value of a thread's chunks, without widening them: among values of which one is not negative the largest
// is the largest as a signed integer, among negative ones the smallest.  Two packed instructions for two 16-bit values (two
// for two of 32 bits with the forms of three operands).  (A NaN may come out or be passed over: its row is NaN anyway.)
template <typename T>
struct LargestOf {
  static constexpr bool HALF = sizeof(T) == 2;
  typedef short i16x2 __attribute__((ext_vector_type(2)));
  using W = typename std::conditional<HALF, i16x2, int>::type;
  W most, least;
  __device__ __forceinline__ void begin(unsigned w) { most = least = __builtin_bit_cast(W, w); }
  __device__ __forceinline__ void add(u32x4 raw) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const W w = __builtin_bit_cast(W, (unsigned)raw[i]);
      most = __builtin_elementwise_max(most, w);
      least = __builtin_elementwise_min(least, w);
    }
  }
  __device__ __forceinline__ float value() const {
    if constexpr (HALF) {
      const short a = most[0] > most[1] ? most[0] : most[1], b = least[0] < least[1] ? least[0] : least[1];
      return to_f32(__builtin_bit_cast(T, a >= 0 ? a : b));
    } else {
      return __builtin_bit_cast(float, most >= 0 ? most : least);
    }
  }
};

// The elements of a chunk that lie outside of the row become -inf: they are below every maximum and their exponential is
// 0, so the passes need no masks.
template <typename T>
__device__ __forceinline__ u32x4 outside_to_minus_infinity(u32x4 raw, int col0, int cols) {
  constexpr int VEC = Chunk<T>::VEC;
  using U = typename std::conditional<sizeof(T) == 2, unsigned short, unsigned>::type;
  const U fill = __builtin_bit_cast(U, from_f32<T>(kNegInf));
  int lo, hi;
  chunk_range<T>(col0, cols, lo, hi);
  U t[VEC];
  __builtin_memcpy(t, &raw, 16);
#pragma unroll
  for (int e = 0; e < VEC; ++e) t[e] = (e >= lo && e < hi) ? t[e] : fill;
  __builtin_memcpy(&raw, t, 16);
  return raw;
}

// The exponentials of 16-bit values are 2^(v log2(e) - c), two instructions and one rounding.  c is a whole number, m log2(e)
// rounded up for an m that is no smaller than the values: it has no rounding of its own, and sums relative to different ones
// are made alike by powers of two.  fp32 takes exp(v - m), whose largest value is exactly 1 (rows of 100 to 65000 differ from 64
// bits by 6.1e-8 in the norm on average, by 8.3e-8 the other way), in three passes: it has half the arithmetic for a byte.
constexpr float kLog2E = 1.44269504088896340736f, kFar = 94548.0f;  // 2^16 log2(e), rounded down
template <typename T>
struct Exponential {
  static constexpr bool SCALED = sizeof(T) == 2;
  float c;  // (SCALED) or the maximum
  __device__ __forceinline__ float operator()(float v) const {
    if constexpr (SCALED)
      return __builtin_amdgcn_exp2f(__builtin_fmaf(v, kLog2E, -c));
    else
      return __expf(v - c);
  }
};
// The power of two for a whole e that is not positive, or infinite or no number where the row's largest value is infinite.  (A sum
// of exponentials, at most 2^17, is 0 from 2^-167 on.)
__host__ __device__ constexpr int power_of_2(float e) { return e > -512.0f ? (int)e : -512; }
static_assert(power_of_2(-0.0f) == 0 && power_of_2(-511.0f) == -511 && power_of_2(-2.0f * kFar) == -512 &&
                  power_of_2(-3.0e38f) == -512 && power_of_2(kNegInf) == -512 && power_of_2(__builtin_nanf("")) == -512,
              "defined for every difference of two scales");
__device__ __forceinline__ float times_power_of_2(float s, float e) { return __builtin_ldexpf(s, power_of_2(e)); }

template <typename T>
__device__ __forceinline__ u32x4 relative_to(u32x4 raw, float m) {
  constexpr int VEC = Chunk<T>::VEC;
  T t[VEC];
  __builtin_memcpy(t, &raw, 16);
#pragma unroll
  for (int e = 0; e < VEC; ++e) t[e] = from_f32<T>(to_f32(t[e]) - m);
  __builtin_memcpy(&raw, t, 16);
  return raw;
}

// Memory, not arithmetic, should decide how long this takes, and a row's loads, arithmetic and stores follow one another,
// with two long rows to a compute unit that do so in step.  So the sum of 16-bit rows is formed while the chunks arrive, each
// thread's relative to the largest value it has seen; what is left behind the last one is a single meeting of the wavefronts,
// and the second exponential beside the stores.  16 vector instructions an element (15 without masks), 21 (18) with the maximum,
// the sum and the results in three passes that each widen, and exponentials of differences; vector units 81 % busy, 94 % then.
// 1024 x 50257 bf16, in and out of HBM: 47.7 -> 44.9 us, 42.0 with streaming stores (4.9 TB/s); 512 rows of it, all resident at
// once, 26.8 -> 20.6; 64 x 8192 3.4 -> 2.9; 6 x 19018 fp16 5.7 -> 4.5.  (One workgroup to a compute unit that requests its next row
// before it works on the one it has: 53 us; half the wavefronts cost more than the order gives.)
template <typename T, int NT, int R, bool RAGGED, bool STREAM>
__global__ void __launch_bounds__(NT, R <= 8 ? 8 : 4) softmax_in_workgroup_kernel(const RowParams p) {
  constexpr int VEC = Chunk<T>::VEC, NW = NT / 64;
  constexpr bool ONLINE = Exponential<T>::SCALED;
  constexpr int G = !ONLINE ? R : R >= 2 ? 2 : 1;  // chunks that share a step of the running maximum
  __shared__ float red[4][NW];
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const long long row = blockIdx.x;
  const T* xr = reinterpret_cast<const T*>(p.x) + row * p.ldx;
  T* yr = reinterpret_cast<T*>(p.y) + row * p.ldy;
  const int shift = RAGGED ? row_shift(p, yr) : 0;
  const int cols_end = p.cols + shift;  // (chunks r * NT .. of the threads are needed if they begin before it: uniform)
  auto col_of = [&](int r) { return (r * NT + tid) * VEC - shift; };
  auto needed = [&](int r) { return r * NT * VEC < cols_end; };
  u32x4 raw[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    raw[r] = u32x4{0u, 0u, 0u, 0u};
    if (needed(r)) raw[r] = load_raw<T>(xr, col_of(r), p.cols);
  }
  auto sum_of = [&](int r, Exponential<T> exponential, float s) {
    float v[VEC];
    widen_chunk<T>(raw[r], v);
#pragma unroll
    for (int e = 0; e < VEC; ++e) s += exponential(v[e]);
    return s;
  };
  // the passes must not share widened values or exponentials: what is kept in registers would double
  auto forget = [&]() {
#pragma unroll
    for (int r = 0; r < R; ++r) asm volatile("" : "+v"(raw[r]));
  };
  float c = -kFar, s = 0.0f;
#pragma unroll
  for (int r0 = 0; r0 < R; r0 += G) {
    if (needed(r0)) {
      LargestOf<T> largest;
#pragma unroll
      for (int r = r0; r < r0 + G; ++r) {
        if (r == r0 || needed(r)) {
          const int col0 = col_of(r);
          // (a wavefront with a chunk that sticks out: one or two of a row's)
          if (__builtin_amdgcn_ballot_w64(col0 < 0 || col0 + VEC > p.cols) != 0)
            raw[r] = outside_to_minus_infinity<T>(raw[r], col0, p.cols);
          if (r == r0) largest.begin(raw[r][0]);
          largest.add(raw[r]);
        }
      }
      if constexpr (ONLINE) {
        const float next = fmaxf(c, __builtin_ceilf(largest.value() * kLog2E));
        if (r0 > 0) s = times_power_of_2(s, c - next);
        c = next;
#pragma unroll
        for (int r = r0; r < r0 + G; ++r)
          if (r == r0 || needed(r)) s = sum_of(r, {c}, s);
      } else {
        c = across_wavefronts<NW, true>(red[0], lane, wave, group_max<64>(largest.value()));
      }
    }
  }
  forget();
  if constexpr (ONLINE) {
    const float cw = group_max<64>(c);
    s = group_sum<64>(times_power_of_2(s, c - cw));
    if (lane == 0) {
      red[0][wave] = cw;
      red[1][wave] = s;
    }
    __syncthreads();
    const float of_wave = red[0][lane % NW];
    c = over_lanes<NW, true>(of_wave);
    s = over_lanes<NW, false>(times_power_of_2(red[1][lane % NW], of_wave - c));
    // Rows whose largest value is farther from zero, infinite ones among them, are made relative to it first: of values of
    // that size any two that differ do so by 256 or more, so that only the zeros of the rounded differences are seen again.
    // (One decision for the whole workgroup.)
    const float c0 = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, c)));
    if (!(__builtin_fabsf(c0) < kFar)) {
      LargestOf<T> largest;
      largest.begin(raw[0][0]);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (needed(r)) largest.add(raw[r]);
      const float m = across_wavefronts<NW, true>(red[2], lane, wave, group_max<64>(largest.value()));
      c = 0.0f;
      s = 0.0f;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (needed(r)) {
          raw[r] = relative_to<T>(raw[r], m);
          s = sum_of(r, {c}, s);
        }
      }
      s = across_wavefronts<NW, false>(red[3], lane, wave, group_sum<64>(s));
      forget();
    }
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (needed(r)) s = sum_of(r, {c}, s);
    forget();
    s = across_wavefronts<NW, false>(red[1], lane, wave, group_sum<64>(s));
  }
  const float inv = 1.0f / s;
  const Exponential<T> exponential{c};
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int col0 = col_of(r);
    if (col0 < p.cols) {
      float v[VEC];
      widen_chunk<T>(raw[r], v);
#pragma unroll
      for (int e = 0; e < VEC; ++e) v[e] = exponential(v[e]) * inv;
      store_chunk<T, RAGGED, STREAM>(yr, col0, p.cols, v);
    }
  }
}

// ---- very long rows: one workgroup per row, streamed ---------------------------------------------------------
// Merge of two (max, sum-of-exp-relative-to-max) pairs; pairs with max = -inf carry sum 0.
__device__ __forceinline__ void merge(float& m, float& s, float m2, float s2) {
  const float mm = fmaxf(m, m2);
  const float a = (m == kNegInf) ? 0.0f : s * __expf(m - mm);
  const float b = (m2 == kNegInf) ? 0.0f : s2 * __expf(m2 - mm);
  m = mm;
  s = a + b;
}

// U chunks of a thread are requested together.
template <typename T, int NT, int U, bool RAGGED, bool SOFTMAX>
__global__ void __launch_bounds__(NT) long_rows_kernel(const RowParams p) {
  constexpr int VEC = Chunk<T>::VEC, NW = NT / 64;
  __shared__ float red_m[NW], red_s[NW];
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const bool is_max = SOFTMAX || p.op == HIDET_REDUCE_MAX;
  const float fill = is_max ? kNegInf : 0.0f;
  const int chunks = p.cols / VEC + (p.cols % VEC != 0);
  for (long long row = blockIdx.x; row < p.rows; row += gridDim.x) {
    const T* xr = reinterpret_cast<const T*>(p.x) + row * p.ldx;
    float m = fill, s = 0.0f;
    for (int c0 = 0; c0 < chunks; c0 += U * NT) {
      u32x4 raw[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + u * NT + tid;
        raw[u] = load_raw<T>(xr, (c < chunks ? c : 0) * VEC, p.cols);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + u * NT + tid;
        if (c >= chunks) continue;
        float v[VEC];
        widen_masked<T, RAGGED>(raw[u], c * VEC, p.cols, !RAGGED, fill, v);
        if (is_max) {
          float cm = v[0];
#pragma unroll
          for (int e = 1; e < VEC; ++e) cm = fmaxf(cm, v[e]);
          if constexpr (SOFTMAX) {
            if (cm != kNegInf) {
              float cs = 0.0f;
#pragma unroll
              for (int e = 0; e < VEC; ++e) cs += __expf(v[e] - cm);
              merge(m, s, cm, cs);
            }
          } else {
            m = fmaxf(m, cm);
          }
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) s += v[e];
        }
      }
    }
    // wavefront, then workgroup
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const float m2 = __shfl_xor(m, o, 64), s2 = __shfl_xor(s, o, 64);
      if constexpr (SOFTMAX)
        merge(m, s, m2, s2);
      else {
        m = fmaxf(m, m2);
        s += s2;
      }
    }
    __syncthreads();  // the previous row's readers are done with red_*
    if (lane == 0) {
      red_m[wave] = m;
      red_s[wave] = s;
    }
    __syncthreads();
    // (in a tree, as in the kernel above)
    float mw[NW], sw[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      mw[w] = red_m[w];
      sw[w] = red_s[w];
    }
#pragma unroll
    for (int n = NW / 2; n >= 1; n /= 2)
#pragma unroll
      for (int w = 0; w < n; ++w) {
        if constexpr (SOFTMAX)
          merge(mw[w], sw[w], mw[w + n], sw[w + n]);
        else {
          mw[w] = fmaxf(mw[w], mw[w + n]);
          sw[w] += sw[w + n];
        }
      }
    m = mw[0];
    s = sw[0];
    if constexpr (SOFTMAX) {
      const float inv = 1.0f / s;
      T* yr = reinterpret_cast<T*>(p.y) + row * p.ldy;
      // (in place: a chunk is written by the thread that reads it, but the last 16 bytes of the row hold elements of
      // two chunks, and the thread that owns the one before may have written its own by then; elements of another
      // chunk are not used)
      for (int c = tid; c < chunks; c += NT) {
        float v[VEC];
        widen_chunk<T>(load_raw<T>(xr, c * VEC, p.cols), v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = __expf(v[e] - m) * inv;
        // (always with the streaming hint: 60 rows of 140000 bf16 28.5 us without, 25.8 with, of 70001 fp32 20.6 and 18.1, one or
        // five of 140000 fp32 28.7 and 28.4; in place there is no difference, nor to a call that reads the results then: the
        // row itself, read twice, has driven out whatever the hint would)
        store_chunk<T, RAGGED, true>(yr, c * VEC, p.cols, v);
      }
    } else if (tid == 0) {
      const float out = is_max ? m : (p.op == HIDET_REDUCE_MEAN ? s / (float)p.cols : s);
      write_scalar(p, row, out, Tag<T>::value);
    }
  }
}

// ---- host side ------------------------------------------------------------------------------------------
constexpr int kMaxBlocks = 256 * 8;  // 8 workgroups of 4 wavefronts fill a compute unit
// The kernel that a problem runs on: decided by its sizes and types, before anything is launched.
enum RowForm { ROWS_PER_WAVEFRONT = 0, ROW_PER_WORKGROUP = 1, ROW_STREAMED = 2 };
struct RowChoice {
  int form;
  int threads;  // that share one row
  int chunks;   // each of them holds (streamed: requests together); 0: a row is shorter than one
};

// Workgroups of `threads` threads that one launch may have: work items are counted in 32 bits (a larger launch is
// refused).  The row-per-workgroup form runs more rows than that in several launches.
constexpr long long max_workgroups(int threads) { return 0xffffffffLL / threads; }

// Outputs of 4 MiB and more, of rows that are not streamed, have the streaming hint where they are not the input: they do not
// stay in the L2s, which otherwise write them back behind the kernel's last store (inputs in HBM, calls one after another: 1024 x
// 50257 bf16 44.4 us without, 41.9 with, 1024 x 33333 fp16 30.5 and 23.3, 1024 x 30000 fp32 52.3 and 46.8, 48828 x 512 fp16 20.0 and
// 16.6; 1024 x 1149 fp16, 2.3 MB, 3.7 and 4.0).  A reader that follows at once has less to find there: with a sum over the
// results the pair takes 0.94 to 1.07 of the time (1024 x 50257 61.4 and 65.3 us, 1024 x 16384 fp16 19.1 and 18.1).  In place the
// lines are in the L2s already, so the hint gains nothing and drives them out: with the sum, 1024 x 50257 56.6 us without, 62.3
// with; attention's chain of three calls, whose softmax works in place, 42 entries of 768 x 768 44.0 and 48.5 us, one of 6144 x
// 6144 66.6 and 76.1.  That ends with what the caches hold: rows of more than 128 KB, one to a compute unit, have left the L2s
// by the time they are stored (rotating buffers, without and with: 502 x 48000 fp32 46.6 and 42.4 us, 749 x 128000 fp16 87.1 and 80.9,
// with the sum 0.98 to 1.03 of the time; 1476 x 65000 with the sum 100.9 and 111.2), and outputs of 256 MiB the last level
// (2129 x 48000 fp32 159.4 and 134.7, with the sum 246 and 219; 4068 x 50257 fp16 150.0 and 128.5; shorter rows 0.99 to 1.03).
template <typename T>
bool streams_output(const RowParams& p) {
  const long long row = (long long)p.cols * (long long)sizeof(T), bytes = p.rows * row;
  return bytes >= (p.x != p.y || row > 128 << 10 ? 4LL << 20 : 256LL << 20);
}

// A softmax whose wavefronts would work on more than eight rows each in turn: with the short butterflies they go in step, all of
// them read and then all of them write, and the lines that two rows share are written at different times.  A workgroup for each few
// rows, spread out by the dispatcher, takes 0.7 to 1.0 of the time where its rows hold 2.5 KB or more (rotating buffers, beside the input,
// in turn -> this way: 919803 x 57 fp16 66.3 -> 43.8 us, 409600 x 128 fp16 37.0 -> 34.2, 104857 x 500 fp16 47.0 -> 37.7, 322236 x 301
// fp32 175.8 -> 133.0, 136533 x 384 fp16 39.9 -> 37.4; in place 39.2 -> 37.7, attention's three calls on 192 entries of 512 x 512
// 93.9 -> 91.8; the worst 1.09, 1248304 x 42 fp16 in place and hot, 38.1 and 41.4).  With less the dispatcher decides
// (4766254 x 11 fp16 130 and 155, 174762 x 300 51.1 and 54.8): these stay in turn and, 32 or more of them to a row, combine
// their lanes through the LDS crossbar, whose queue spreads the wavefronts (646621 x 300 fp16 194.4 us with butterflies, 187.3 so,
// 1426371 x 136 168.3 and 160.0; not 2586487 x 75 245 and 252, 12932437 x 15 497 and 515).
// With fewer rows in turn neither pays: 23437 x 256 one by one 5.3 us, 4.9 in turn, 20000 x 150 fp32 through the crossbar 6.6,
// with butterflies 6.2.  Nor does a workgroup for each few rows in reductions, which write next to nothing.
bool rows_in_turn(long long rows, int lanes) { return rows > 8LL * kMaxBlocks * 4 * (64 / lanes); }
bool spreads_rows(long long rows, long long row_bytes, int lanes) {
  return rows_in_turn(rows, lanes) && 4 * (64 / lanes) * row_bytes >= 2560;
}
// Workgroups of a launch whose wavefronts share a row between `lanes` lanes.
long long wavefront_blocks(bool softmax, long long rows, long long row_bytes, int lanes) {
  const long long per_block = 4 * (64 / lanes), wanted = rows / per_block + (rows % per_block != 0);
  return std::min(wanted, softmax && spreads_rows(rows, row_bytes, lanes) ? max_workgroups(256) : (long long)kMaxBlocks);
}

template <typename T, int L, int R, bool SOFTMAX, bool STREAM, bool CROSSBAR>
hipError_t launch_wavefront_as(const RowParams& p, dim3 grid, hipStream_t stream) {
  if constexpr (R == 0)
    hipLaunchKernelGGL((rows_in_registers_kernel<T, L, 1, SHORT, SOFTMAX, false, false>), grid, dim3(256), 0, stream, p);
  else if (p.cols % Chunk<T>::VEC == 0)
    hipLaunchKernelGGL((rows_in_registers_kernel<T, L, R, WHOLE, SOFTMAX, STREAM, CROSSBAR>), grid, dim3(256), 0, stream, p);
  else if constexpr (R <= 4)  // (longer ragged rows take a workgroup)
    hipLaunchKernelGGL((rows_in_registers_kernel<T, L, R, RAGGED_END, SOFTMAX, STREAM, CROSSBAR>), grid, dim3(256), 0, stream, p);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// (The streaming hint writes lines that two rows share in parts.  Short ragged rows have many of them: beside the input, 112347 x 57
// fp16 13.5 us without, 15.8 with, 149796 x 42 fp32 13.6 and 14.6, 103991 x 121 fp16 13.1 and 13.0, 83886 x 150 18.1 and 17.6.  Ragged
// rows in turn write the parts at different times: 646621 x 300 fp16 187.3 and 193.4, 1293243 x 75 fp32 192.1 and 210.2.)
template <typename T, int L, int R, bool SOFTMAX>
hipError_t launch_wavefront(const RowParams& p, hipStream_t stream) {
  const long long row_bytes = (long long)p.cols * (long long)sizeof(T);
  const dim3 grid((unsigned)wavefront_blocks(SOFTMAX, p.rows, row_bytes, L));
  if constexpr (SOFTMAX && R > 0) {
    const bool in_turn = rows_in_turn(p.rows, L) && !spreads_rows(p.rows, row_bytes, L);
    const bool streams = streams_output<T>(p) && (row_bytes % 16 == 0 || (row_bytes >= 256 && !in_turn));
    if constexpr (R == 1 && L >= 32)  // (more chunks a lane are more than 2.5 KB)
      if (in_turn)
        return streams ? launch_wavefront_as<T, L, R, true, true, true>(p, grid, stream)
                       : launch_wavefront_as<T, L, R, true, false, true>(p, grid, stream);
    if (streams) return launch_wavefront_as<T, L, R, true, true, false>(p, grid, stream);
  }
  // Reductions of ragged 16-bit rows of up to four chunks have more vector instructions than any for a byte: in turn, their lanes
  // meet through the LDS crossbar, beside them (7149381 x 11 fp16 sums 101 us with butterflies, 90 so, 2097152 x 17 31.4 and 28.5, 2536877
  // x 31 36.0 and 34.4; 2383127 x 33 25.9 and 29.1, 279620 x 15, not in turn, 5.5 and 6.4; whole rows 1.1 to 1.2 of the time, fp32 too).
  if constexpr (!SOFTMAX && R == 1 && L == 8 && sizeof(T) == 2) {
    if (row_bytes % 16 != 0 && row_bytes < 64 && rows_in_turn(p.rows, L)) {
      hipLaunchKernelGGL((rows_in_registers_kernel<T, L, R, RAGGED_END, false, false, true>), grid, dim3(256), 0, stream, p);
      return hipGetLastError();
    }
  }
  return launch_wavefront_as<T, L, R, SOFTMAX, false, false>(p, grid, stream);
}

template <typename T, int NT, int R, bool STREAM>
void launch_softmax(const RowParams& q, dim3 grid, bool whole, hipStream_t stream) {
  if (whole)
    hipLaunchKernelGGL((softmax_in_workgroup_kernel<T, NT, R, false, STREAM>), grid, dim3(NT), 0, stream, q);
  else
    hipLaunchKernelGGL((softmax_in_workgroup_kernel<T, NT, R, true, STREAM>), grid, dim3(NT), 0, stream, q);
}

template <typename T, int NT, int R, bool SOFTMAX>
hipError_t launch_workgroup(const RowParams& p, hipStream_t stream) {
  RowParams q = p;
  for (long long row = 0; row < p.rows; row += max_workgroups(NT)) {
    q.x = static_cast<const char*>(p.x) + row * p.ldx * (long long)sizeof(T);
    q.y = static_cast<char*>(p.y) + (SOFTMAX ? row * p.ldy * (long long)sizeof(T) : row * (p.out_f32 ? 4 : (long long)sizeof(T)));
    q.rows = p.rows - row < max_workgroups(NT) ? p.rows - row : max_workgroups(NT);
    const bool whole = p.cols % Chunk<T>::VEC == 0 && !p.shift;
    const dim3 grid((unsigned)q.rows);
    if constexpr (SOFTMAX) {
      if (streams_output<T>(p))
        launch_softmax<T, NT, R, true>(q, grid, whole, stream);
      else
        launch_softmax<T, NT, R, false>(q, grid, whole, stream);
    } else {
      if (whole)
        hipLaunchKernelGGL((reduce_in_workgroup_kernel<T, NT, R, false>), grid, dim3(NT), 0, stream, q);
      else
        hipLaunchKernelGGL((reduce_in_workgroup_kernel<T, NT, R, true>), grid, dim3(NT), 0, stream, q);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T, int NT, int U, bool RAGGED, bool SOFTMAX>
hipError_t launch_streamed(const RowParams& p, hipStream_t stream) {
  const long long blocks = p.rows < kMaxBlocks ? p.rows : kMaxBlocks;
  hipLaunchKernelGGL((long_rows_kernel<T, NT, U, RAGGED, SOFTMAX>), dim3((unsigned)blocks), dim3(NT), 0, stream, p);
  return hipGetLastError();
}

int chunks_of(int elem_size, int cols) { return cols / (16 / elem_size) + (cols % (16 / elem_size) != 0); }

RowChoice choose_rows(int elem_size, bool softmax, long long rows, int cols) {
  const int chunks = chunks_of(elem_size, cols);
  if (cols < 16 / elem_size) return {ROWS_PER_WAVEFRONT, 8, 0};
  if (chunks <= 8) return {ROWS_PER_WAVEFRONT, 8, 1};
  if (chunks <= 16) return {ROWS_PER_WAVEFRONT, 16, 1};
  if (chunks <= 32) return {ROWS_PER_WAVEFRONT, 32, 1};
  if (chunks <= 64) return {ROWS_PER_WAVEFRONT, 64, 1};
  if (chunks <= 128) return {ROWS_PER_WAVEFRONT, 64, 2};
  // Few rows: a workgroup per row has more loads in flight for each of them (200 x 2048 bf16: 3.9 -> 2.9 us).  With
  // thousands of rows the compute units are full either way, and the threads that a row does not fill and the two
  // barriers cost more than they give, so a wavefront per row is faster (65536 x 1152 fp16 softmax: 92 us on 256
  // threads, 50 us on a wavefront; 16384 x 576 fp32 sum 10.8 and 6.7 us) -- up to 384 chunks, where the widened row begins
  // to crowd the registers.  Reductions keep nothing after the sum and gain up to 512 chunks (4096 x 1600 fp32: 5.2 and
  // 3.9 us).  The more rows, the more memory alone decides, which 256 threads use better: up to 320 chunks (65536 x 1400
  // fp32 sum 58 us on 256 threads, 64 us on a wavefront; 65536 x 1200 58 and 49 us), in an fp32 softmax, with half the
  // arithmetic per byte, up to 256 (16384 x 1200: 29.9 and 31.4 us) and then 192 (65536 x 1000: 90 and 100 us, x 768: 79
  // and 75 us).
  // Masks of a ragged length are paid by every lane: there it takes more rows and stops at 256 chunks (1024 x 1149 fp16
  // softmax: 4.2 us on 256 threads, 4.7 us on a wavefront; 4096 rows 9.0 and 7.9 us).
  const bool ragged = cols % (16 / elem_size) != 0;
  int wavefront_chunks = ragged ? 256 : rows >= 16384 ? 320 : softmax || rows > 8192 ? 384 : 512;
  if (softmax && elem_size == 4 && rows >= 16384) wavefront_chunks = rows >= 32768 ? 192 : 256;
  if (rows >= (ragged ? 2048 : 1024) && chunks <= wavefront_chunks)
    return {ROWS_PER_WAVEFRONT, 64, chunks <= 256 ? 4 : 8};
  if (chunks <= 256) return {ROW_PER_WORKGROUP, 256, 1};
  if (chunks <= 512) return {ROW_PER_WORKGROUP, 256, 2};
  // (513 chunks fill half of 512 threads with a second one: 4096 x 2052 fp32 softmax 14.2 us, 12.1 us on 256 threads
  // with up to four each; below 512 rows the other way round, 3.5 and 3.7 us)
  if (chunks <= 768 && rows >= 512) return {ROW_PER_WORKGROUP, 256, 4};
  // A reduction has nothing to keep after the sum.  From 512 rows on, two or more workgroups wait for every compute unit,
  // and ones that stream whole chunks, with no register held for the row, read faster than those that hold it (16-bit
  // rows of 2456 chunks: 1024 of them 8.9 us held by 1024 threads, 7.7 us streamed by 512; 8192 of them 54 and 50 us).
  // Up to 2048 chunks this ends where memory alone decides (1024 rows of 1311 chunks: 4.9 and 4.1 us; 8192: 26.6 and
  // 28.6 us).
  if (!softmax && !ragged && rows >= 512 && chunks > 1024 && (chunks > 2048 || rows <= 2048)) return {ROW_STREAMED, 512, 4};
  // More threads with fewer chunks each are the better split of longer rows (64 x 8192 bf16: 4.0 us on 256 threads, 3.6
  // us on 512), too many leave most of them idle (4096 x 8200: 28 us on 512 threads, 39 us on 1024).
  if (chunks <= 1024) return {ROW_PER_WORKGROUP, 512, 2};
  if (chunks <= 2048) return {ROW_PER_WORKGROUP, 512, 4};
  if (chunks <= 4096) return {ROW_PER_WORKGROUP, 1024, 4};
  if (chunks < 8192) return {ROW_PER_WORKGROUP, 1024, 8};
  // (ragged rows: the masks take registers, two chunks in flight are enough; 1024 rows of 10000 16-bit chunks 29 us, held
  // 33 us)
  if (!softmax && rows >= 512) return {ROW_STREAMED, 512, 2};
  if (chunks <= 16384) return {ROW_PER_WORKGROUP, 1024, 16};
  // (the most threads and bytes in flight for one row: 90 x 500000 bf16 94 us, 143 us on 512 threads)
  return {ROW_STREAMED, 1024, 4};
}

constexpr int choice_key(int form, int threads, int chunks) { return (form * 2048 + threads) * 32 + chunks; }

template <typename T, bool SOFTMAX>
hipError_t dispatch(const RowParams& p_in, hipStream_t stream) {
  RowParams p = p_in;
  const int chunks = chunks_of(sizeof(T), p.cols);
  // the shifted grid needs room for one chunk more, and costs a few element-wise stores at both ends of a row
  if (chunks <= 4096 || chunks >= 16384) p.shift = 0;
  const RowChoice c = choose_rows(sizeof(T), SOFTMAX, p.rows, p.cols);
  switch (choice_key(c.form, c.threads, c.chunks)) {
    case choice_key(ROWS_PER_WAVEFRONT, 8, 0): return launch_wavefront<T, 8, 0, SOFTMAX>(p, stream);
    case choice_key(ROWS_PER_WAVEFRONT, 8, 1): return launch_wavefront<T, 8, 1, SOFTMAX>(p, stream);
    case choice_key(ROWS_PER_WAVEFRONT, 16, 1): return launch_wavefront<T, 16, 1, SOFTMAX>(p, stream);
    case choice_key(ROWS_PER_WAVEFRONT, 32, 1): return launch_wavefront<T, 32, 1, SOFTMAX>(p, stream);
    case choice_key(ROWS_PER_WAVEFRONT, 64, 1): return launch_wavefront<T, 64, 1, SOFTMAX>(p, stream);
    case choice_key(ROWS_PER_WAVEFRONT, 64, 2): return launch_wavefront<T, 64, 2, SOFTMAX>(p, stream);
    case choice_key(ROWS_PER_WAVEFRONT, 64, 4): return launch_wavefront<T, 64, 4, SOFTMAX>(p, stream);
    case choice_key(ROWS_PER_WAVEFRONT, 64, 8): return launch_wavefront<T, 64, 8, SOFTMAX>(p, stream);
    case choice_key(ROW_PER_WORKGROUP, 256, 1): return launch_workgroup<T, 256, 1, SOFTMAX>(p, stream);
    case choice_key(ROW_PER_WORKGROUP, 256, 2): return launch_workgroup<T, 256, 2, SOFTMAX>(p, stream);
    case choice_key(ROW_PER_WORKGROUP, 256, 4): return launch_workgroup<T, 256, 4, SOFTMAX>(p, stream);
    case choice_key(ROW_PER_WORKGROUP, 512, 2): return launch_workgroup<T, 512, 2, SOFTMAX>(p, stream);
    case choice_key(ROW_PER_WORKGROUP, 512, 4): return launch_workgroup<T, 512, 4, SOFTMAX>(p, stream);
    case choice_key(ROW_PER_WORKGROUP, 1024, 4): return launch_workgroup<T, 1024, 4, SOFTMAX>(p, stream);
    case choice_key(ROW_PER_WORKGROUP, 1024, 8): return launch_workgroup<T, 1024, 8, SOFTMAX>(p, stream);
    case choice_key(ROW_PER_WORKGROUP, 1024, 16): return launch_workgroup<T, 1024, 16, SOFTMAX>(p, stream);
    case choice_key(ROW_STREAMED, 1024, 4): return launch_streamed<T, 1024, 4, true, SOFTMAX>(p, stream);
    default: break;
  }
  if constexpr (!SOFTMAX) switch (choice_key(c.form, c.threads, c.chunks)) {  // (without masks: chosen for whole rows only)
    case choice_key(ROW_STREAMED, 512, 2): return launch_streamed<T, 512, 2, true, SOFTMAX>(p, stream);
    case choice_key(ROW_STREAMED, 512, 4): return launch_streamed<T, 512, 4, false, SOFTMAX>(p, stream);
    default: break;
  }
  return hipErrorInvalidValue;  // (a choice that is not built)
}

template <bool SOFTMAX>
hipError_t dispatch_dtype(int dtype, const RowParams& p, hipStream_t stream) {
  switch (dtype) {
    case HIDET_F32: return dispatch<float, SOFTMAX>(p, stream);
    case HIDET_F16: return dispatch<f16, SOFTMAX>(p, stream);
    default: return dispatch<bf16, SOFTMAX>(p, stream);
  }
}

bool aligned_to(const void* ptr, size_t a) { return (reinterpret_cast<uintptr_t>(ptr) % a) == 0; }
int elem_bytes(int dtype) { return dtype == HIDET_F32 ? 4 : 2; }

}  // namespace

// rows * ld elements must be addressable (below 2^47), so that the 64-bit row offsets cannot overflow
static bool span_ok(long long rows, long long ld) {
  constexpr long long lim = 1LL << 47;
  return ld <= lim && (rows <= 1 || ld <= lim / rows);
}

extern "C" {

hidet_status_t hidet_row_schedule(int32_t dtype, int32_t softmax, int64_t rows, int64_t cols, hidet_row_schedule_t* out) {
  if (dtype < 0 || dtype > 2 || rows <= 0 || cols < 0 || !out) return HIDET_ERR_INVALID_ARG;
  if (cols > 0x7fffffffLL - 64) return HIDET_ERR_UNSUPPORTED;
  const RowChoice c = choose_rows(elem_bytes(dtype), softmax != 0, rows, (int)cols);
  out->form = c.form;
  out->threads_per_row = c.threads;
  out->chunks_per_thread = c.chunks;
  out->workgroup_size = c.form == ROWS_PER_WAVEFRONT ? 256 : c.threads;
  const long long rows_per_workgroup = out->workgroup_size / c.threads;
  const long long limit = c.form == ROW_PER_WORKGROUP ? max_workgroups(c.threads) : kMaxBlocks;
  const long long wanted = (rows - 1) / rows_per_workgroup + 1;
  out->workgroups = c.form == ROWS_PER_WAVEFRONT
                        ? wavefront_blocks(softmax != 0, rows, cols * elem_bytes(dtype), c.threads)
                        : std::min(wanted, limit);
  out->launches = c.form == ROW_PER_WORKGROUP ? (wanted - 1) / limit + 1 : 1;
  return HIDET_OK;
}

hidet_status_t hidet_reduce_rows(int32_t in, int32_t out, int32_t op, int64_t rows, int64_t cols, const void* x,
                                 int64_t ldx, void* y, void* stream) {
  if (in < 0 || in > 2 || out < 0 || out > 2 || op < 0 || op > 2) return HIDET_ERR_INVALID_ARG;
  if (out != in && out != HIDET_F32) return HIDET_ERR_UNSUPPORTED;
  if (rows < 0 || cols < 0) return HIDET_ERR_INVALID_ARG;
  if (cols > 0x7fffffffLL - 64) return HIDET_ERR_UNSUPPORTED;
  if (rows == 0) return HIDET_OK;
  if (!y || (cols > 0 && !x) || ldx < cols) return HIDET_ERR_INVALID_ARG;
  if (!span_ok(rows, ldx)) return HIDET_ERR_UNSUPPORTED;
  if (!aligned_to(x, (size_t)elem_bytes(in)) || !aligned_to(y, (size_t)elem_bytes(out))) return HIDET_ERR_ALIGNMENT;
  RowParams p;
  p.x = x;
  p.y = y;
  p.ldx = ldx;
  p.ldy = 0;
  p.rows = rows;
  p.cols = (int)cols;
  p.op = op;
  p.out_f32 = out == HIDET_F32 ? 1 : 0;
  p.shift = 0;
  return dispatch_dtype<false>(in, p, (hipStream_t)stream) == hipSuccess ? HIDET_OK : HIDET_ERR_LAUNCH;
}

hidet_status_t hidet_softmax_rows(int32_t dtype, int64_t rows, int64_t cols, const void* x, int64_t ldx, void* y,
                                  int64_t ldy, void* stream) {
  if (dtype < 0 || dtype > 2) return HIDET_ERR_INVALID_ARG;
  if (rows < 0 || cols < 0) return HIDET_ERR_INVALID_ARG;
  if (cols > 0x7fffffffLL - 64) return HIDET_ERR_UNSUPPORTED;
  if (rows == 0 || cols == 0) return HIDET_OK;
  if (!x || !y || ldx < cols || ldy < cols) return HIDET_ERR_INVALID_ARG;
  if (!span_ok(rows, ldx) || !span_ok(rows, ldy)) return HIDET_ERR_UNSUPPORTED;
  const size_t es = (size_t)elem_bytes(dtype);
  if (!aligned_to(x, es) || !aligned_to(y, es)) return HIDET_ERR_ALIGNMENT;
  RowParams p;
  p.x = x;
  p.y = y;
  p.ldx = ldx;
  p.ldy = ldy;
  p.rows = rows;
  p.cols = (int)cols;
  p.op = HIDET_REDUCE_MAX;
  p.out_f32 = 0;
  p.shift = (aligned_to(y, 16) && ldy % (16 / (int)es) == 0) ? 0 : 1;
  return dispatch_dtype<true>(dtype, p, (hipStream_t)stream) == hipSuccess ? HIDET_OK : HIDET_ERR_LAUNCH;
}

}  // extern "C"

// The K-splitting schedule of small output tiles: every wavefront streams its own share of K.
//
// A problem with few output tiles is bound by the chain of one workgroup, not by throughput: with the K tiles shared by
// all wavefronts (gemm_kernel) each of them is a round trip to memory, an LDS write, a barrier and the dependent
// fragment reads.  Here nothing is shared before the end.  K is consumed in steps; wavefront w owns the steps w, w + 8, ...
// of the whole BM x BN tile, fetches them with direct global -> LDS loads into a ring of its own (D steps in flight, waited
// for by count), and multiplies them without meeting another wavefront.  The partial tiles meet in LDS once, where each
// group of four outputs is summed in wavefront order and stored.
//
// What bounds it is the chain itself: at 128x768x3072 a wavefront issues one instruction in 17 clocks of its 18 thousand (of the
// kernel's 19), and the first-level cache of a compute unit takes 4800 accesses, a quarter of the clocks at one a clock.  That
// part decides the width of a step: 64 values of k on tiles up to 32x32, a whole line of every row of a K-contiguous operand, with
// eight wavefronts; with steps of 32 and sixteen wavefronts, which keep as many bytes in flight, 8x3072x768 on 16x32 tiles
// takes 5.0 us instead of 4.3, 128x768x3072 9.1 instead of 8.5.  On the larger tiles, whose LDS has no room for two steps of
// 64 and eight wavefronts, steps of 32 and eight wavefronts win over steps of 64 and four (1024^3 on 64x64: 9.3 and 10.7 us).
// Against the shared K tiles (microseconds in a replayed graph): aligned rows 8x3072x768 5.4 -> 4.3, 8x768x3072 7.6 -> 7.1,
// 128x768x3072 9.3 -> 8.5, 200x512x2048 on 32x32 7.9 -> 6.6; element-aligned ones, which the general schedule fetches
// through registers under predicates, 37x82x2658 14.0 -> 5.7, 80x45x796 6.1 -> 4.7.  Empty kernels take 1.5 there, and
// the shortest chain of a product about 3.3.
//
// A last step that K ends in takes part in a ring with zeros in the place of the chunks outside.  Where rows are only
// element aligned, the last step goes through registers, whole or not (no 16-byte access then touches the last row of an
// M/N-contiguous operand); it is requested before the loop, so that it is there when its wavefront comes to it.
#pragma once

#include "epilogue.hpp"

namespace hidet {

// The same tile with wavefronts that stream K (Cfg describes the tile as the general schedule runs it).
template <class Cfg>
struct WaveStream {
  static constexpr int BM = Cfg::BM, BN = Cfg::BN;
  static constexpr int STEP = BM * BN > 32 * 32 ? 32 : 64;
  static constexpr bool BUILT = Cfg::SCHED == SCHED_KSPLIT && !Cfg::IS_F32 && Cfg::MI == 16 && BM <= 64 && BN <= 64 && !Cfg::GATHER_B;
  static constexpr int NW = 8;
  static constexpr int NT = NW * 64;
  static constexpr int A_BYTES = BM * STEP * 2, B_BYTES = BN * STEP * 2, STEP_BYTES = A_BYTES + B_BYTES;
  static constexpr int FIT = 144 * 1024 / (NW * STEP_BYTES);
  static constexpr int D = FIT > 4 ? 4 : FIT;  // steps of a wavefront's ring
  static constexpr int RING_BYTES = D * STEP_BYTES;
  static constexpr int PART_BYTES = BM * (BN * 4 + 16);  // (PartialTiles)
  static constexpr int LDS_BYTES = NW * (RING_BYTES > PART_BYTES ? RING_BYTES : PART_BYTES);
  static_assert(!BUILT || (D >= 2 && LDS_BYTES <= 160 * 1024), "a ring of two steps at least, in the LDS of a compute unit");
};

// at most N vector memory operations in flight
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "6-bit counter");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <class Frag>
__device__ __forceinline__ Frag relu_fragment(Frag f) {  // (a negative value is negative as an integer: Operand::store)
  typedef short i16x8 __attribute__((ext_vector_type(8)));
  const i16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
  return __builtin_bit_cast(Frag, __builtin_elementwise_max(__builtin_bit_cast(i16x8, f), z));
}

// ---- the fused epilogue of a group of four columns, in two parts -- what it reads, what it computes and stores (store4
// does both at the end, where the large tiles, short of registers, want them) ------------------------------------------
template <typename TO>
struct __attribute__((packed, aligned(sizeof(TO)))) GroupOf4 {  // one access; the address need only be element aligned
  TO e[4];
};

// The residual of a group, widened (zeros where there is none): a kernel that is bound by one latency chain asks for it
// before its main loop.  `row`: offset of the group's row, `ccol`: of its first column.
template <typename TO>
__device__ __forceinline__ void load_residual4(const GemmParams& p, const TO* __restrict__ R, long long row, int n, long long ccol,
                                               int nvalid, float (&res)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) res[e] = 0.0f;
  if (R == nullptr || nvalid <= 0) return;
  const long long roff = row + ccol;
  if (p.vec_store && nvalid == 4) {
    TO r[4];
    *reinterpret_cast<GroupOf4<TO>*>(r) = *reinterpret_cast<const GroupOf4<TO>*>(R + roff);
#pragma unroll
    for (int e = 0; e < 4; ++e) res[e] = to_f32(r[e]);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (e < nvalid) {
        long long ro = roff + e;
        if (p.out_map != 0) ro = row + col_offset<MAP_PLAIN>(p, n + e);
        res[e] = to_f32(R[ro]);
      }
    }
  }
}

// The group's results from its sums, biases and residual.
template <typename TO>
__device__ __forceinline__ void finish4(const GemmParams& p, TO* __restrict__ C, const float (&bias)[4], const float (&res)[4],
                                        bool residual, long long row, int n, long long ccol, int nvalid, const float (&acc)[4]) {
  if (nvalid <= 0) return;
  const long long off = row + ccol;
  const bool whole = p.vec_store && nvalid == 4;
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = p.alpha * acc[e] + bias[e];  // zeros where there is no bias
  if (residual) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += res[e];
  }
  if (p.relu) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = v[e] < 0.0f ? 0.0f : v[e];
  }
  TO o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = from_f32<TO>(v[e]);
  if (whole) {
    // the output is not read again by this kernel: streamed, or written through the die's L2 (see store_group)
    if (p.vec_store >= 2) {  // 4-element aligned address
      if constexpr (sizeof(TO) == 2)
        store_group(C + off, o, p.vec_store == 3);
      else
        __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(o), reinterpret_cast<u32x4*>(C + off));
    } else {
      *reinterpret_cast<GroupOf4<TO>*>(C + off) = *reinterpret_cast<const GroupOf4<TO>*>(o);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (e < nvalid) {
        long long oo = off + e;
        if (p.out_map != 0) oo = row + col_offset<MAP_PLAIN>(p, n + e);
        C[oo] = o[e];
      }
    }
  }
}

// ---- the end of a kernel whose wavefronts hold a partial tile each: they meet in LDS, where each group of four outputs is summed
// in wavefront order and stored --------------------------------------------------------------------------------------------
template <typename TO, int BM, int BN, int NW>
struct PartialTiles {
  static constexpr int NT = NW * 64, FM = BM / 16, FN = BN / 16;
  static constexpr int ROW_BYTES = BN * 4 + 16;  // rows start 4 banks apart
  static constexpr int PART_BYTES = BM * ROW_BYTES;
  // a thread finishes groups of four columns: `tid`, `tid` + NT, ... in row-major order over the tile
  static constexpr int GROUPS = BM * BN / 4, PER_ROW = BN / 4, PASSES = (GROUPS + NT - 1) / NT;
  static_assert(NT % PER_ROW == 0, "a thread keeps its columns");
  int c4, col, valid;
  long long ccol;
  TO* C;
  const TO* R;
  float bias[PASSES][4], res[PASSES][4];
  long long row_at[PASSES];  // offset of the group's row in C; negative: no row of C

  // what the end needs from memory, requested ahead of it
  __device__ __forceinline__ void request(const GemmParams& p, const BlockCoords& bc) {
    c4 = (int)threadIdx.x % PER_ROW;
    col = bc.n0 + c4 * 4;
    C = reinterpret_cast<TO*>(p.C) + (long long)bc.cbatch * p.strideC;
    R = p.residual ? reinterpret_cast<const TO*>(p.residual) + (long long)bc.batch * p.strideR : nullptr;
    const TO* bias_ptr = reinterpret_cast<const TO*>(p.bias);
    ccol = col_offset<MAP_PLAIN>(p, col);
    valid = group_valid<MAP_PLAIN>(p, col);
#pragma unroll
    for (int s = 0; s < PASSES; ++s) {
      const int g = s * NT + (int)threadIdx.x, m = bc.m0 + g / PER_ROW;
      row_at[s] = g < GROUPS && m < p.M ? row_offset<MAP_PLAIN>(p, m, p.ldc) : -1;
      asm volatile("" : "+v"(row_at[s]));  // (now, while the first step is on its way, not at the end)
#pragma unroll
      for (int e = 0; e < 4; ++e) bias[s][e] = res[s][e] = 0.0f;
      if (g < GROUPS && m < p.M) {
        if (p.bias_axis != 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (p.bias_axis == 2 || e < valid) bias[s][e] = to_f32(bias_ptr[p.bias_axis == 2 ? m : col + e]);
        }
        load_residual4<TO>(p, R, p.out_map != 0 ? row_at[s] : (long long)m * p.ldr, col, ccol, valid, res[s]);
      }
    }
  }

  // (of zeros from a wavefront that had no step).  PAIRS: fragments 2 j and 2 j + 1 hold the even and the odd ones of 32 columns.
  template <bool PAIRS = false>
  __device__ __forceinline__ void finish(const GemmParams& p, const f32x4 (&acc)[FM][FN], unsigned char* smem, int wave, int lane) {
    unsigned char* part = smem + wave * PART_BYTES;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      unsigned char* row = part + (i * 16 + lane % 16) * ROW_BYTES;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        if constexpr (PAIRS) {
          const f32x4 even = acc[i][j & ~1], odd = acc[i][j | 1];
          const int r = 2 * (j & 1);
          const int at = (j & ~1) * 16 + 8 * (lane / 16) + 4 * (j & 1);
          *reinterpret_cast<f32x4*>(row + at * 4) = f32x4{even[r], odd[r], even[r + 1], odd[r + 1]};
        } else {
          *reinterpret_cast<f32x4*>(row + (j * 16 + 4 * (lane / 16)) * 4) = acc[i][j];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < PASSES; ++s) {
      if (row_at[s] >= 0) {
        const int row = (s * NT + (int)threadIdx.x) / PER_ROW;
        const unsigned char* src = smem + row * ROW_BYTES + c4 * 16;
        f32x4 v[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) v[w] = *reinterpret_cast<const f32x4*>(src + w * PART_BYTES);
        f32x4 sum = v[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += v[w];
        const float out[4] = {sum[0], sum[1], sum[2], sum[3]};
        finish4<TO>(p, C, bias[s], res[s], R != nullptr, row_at[s], col, ccol, valid, out);
      }
    }
  }
};

// ---- the last step of K on element-aligned rows, through registers ----------------------------------------------------------
// Requested without a branch and finished when it is stored, so that nothing waits for it in between (under the predicates of
// the general schedule instead, 80x45x796 on 16x16 tiles takes 4.9 us, not 4.7): a chunk that sticks out of the operand's end
// is read as the last 16 bytes of the operand and shifted down afterwards.  Along M/N what lies past the edge only reaches
// outputs that are never stored; along K it becomes zero.
template <class Op, int LAYOUT>
struct TailStep {
  static_assert(Op::VEC == 8, "16-bit types");
  u32x4 raw[Op::NL];
  int keep[Op::NL], down[Op::NL];  // elements that lie inside K; by how many elements the chunk is to be shifted down

  __device__ __forceinline__ void request(const Op& op, int lane, int k0) {
#pragma unroll
    for (int q = 0; q < Op::NL; ++q) {
      const tmap::Task t = Op::LoadMap::task(lane, q);
      const int sr = t.i, sc = t.j * 8;
      if (op.span < 8) {  // (uniform: an operand of less than 16 bytes)
        raw[q] = op.gather(sr, sc, k0);
        keep[q] = 8;
        down[q] = 0;
        continue;
      }
      long long base;
      int inside;
      if constexpr (LAYOUT == L_KC) {
        base = (long long)(sr < op.rows_left ? sr : op.rows_left - 1) * op.ld + (k0 + sc);
        inside = op.K - (k0 + sc);
      } else {
        base = (long long)(k0 + sr) * op.ld + (sc < op.rows_left ? sc : 0);
        inside = k0 + sr < op.K ? 8 : 0;
      }
      if (inside <= 0) base = 0;
      const long long over = base + 8 - op.span;
      down[q] = over > 0 ? (int)over : 0;
      keep[q] = inside < 0 ? 0 : (inside > 8 ? 8 : inside);
      raw[q] = reinterpret_cast<const typename Op::Unaligned*>(op.src + (base - down[q]))->v;
    }
  }

  __device__ __forceinline__ void store(const Op& op, int lane, unsigned char* tile) {
#pragma unroll
    for (int q = 0; q < Op::NL; ++q) {
      u32x4 v = raw[q];
      const int d = down[q], n = keep[q];
      if (d & 4) v = u32x4{v[2], v[3], 0u, 0u};
      if (d & 2) v = u32x4{v[1], v[2], v[3], 0u};
      if (d & 1) v = u32x4{(v[0] >> 16) | (v[1] << 16), (v[1] >> 16) | (v[2] << 16), (v[2] >> 16) | (v[3] << 16), v[3] >> 16};
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] &= n >= 2 * i + 2 ? 0xffffffffu : (n == 2 * i + 1 ? 0x0000ffffu : 0u);
      raw[q] = v;
    }
    op.store(raw, lane, tile);
  }
};

template <class Cfg, class Params>
__global__ void __launch_bounds__(WaveStream<Cfg>::NT) gemm_kernel_waves(const Params params) {
  const GemmParams& p = whole_params<Cfg::BM, Cfg::BN>(params);
  using S = WaveStream<Cfg>;
  using T = typename Cfg::T;
  using TO = typename Cfg::TO;
  constexpr int BM = S::BM, BN = S::BN, STEP = S::STEP, NW = S::NW, D = S::D, KS = STEP / 32, FM = BM / 16, FN = BN / 16;
  constexpr bool ELEM = Cfg::MODE_A == LD_ELEM;
  static_assert(Cfg::MODE_A == Cfg::MODE_B && Cfg::MAPPER == MAP_PLAIN, "plain GEMM operands");
  // one wavefront loads a whole step
  using OpA = Operand<T, BM, STEP, Cfg::LA, Cfg::MODE_A, 64, 16>;
  using OpB = Operand<T, BN, STEP, Cfg::LB, Cfg::MODE_B, 64, 16>;
  constexpr int LOADS = OpA::NL + OpB::NL;  // direct loads of a step
  static_assert(D * LOADS < 64, "the loads in flight are counted in six bits");

  __shared__ __attribute__((aligned(16))) unsigned char smem[S::LDS_BYTES];

  const int lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const BlockCoords bc = block_coords<BM, BN>(p);
  OpA opa;
  OpB opb;
  setup_operands<Cfg>(p, bc, opa, opb);

  // ---- steps by direct loads: the whole ones, without the last one where rows are only element aligned
  const int whole = ELEM ? (bc.k_len > 0 ? (bc.k_len - 1) / STEP : 0) : bc.k_len / STEP;
  const int mine = whole > wave ? (whole - wave + NW - 1) / NW : 0;
  const bool tail = whole * STEP < bc.k_len && wave == whole % NW;  // this wavefront multiplies the last step
  const int n = mine + (!ELEM && tail ? 1 : 0);                      // steps of its ring
  unsigned char* ring = smem + wave * S::RING_BYTES;
  const unsigned ring_lds = (unsigned)(size_t)(__attribute__((address_space(3))) void*)ring;
  opa.init_direct(lane, ELEM);
  opb.init_direct(lane, ELEM);
  auto request = [&](int i, int slot) {  // this wavefront's step i
    const int k0 = (wave + i * NW) * STEP;
    const unsigned at = ring_lds + (unsigned)(slot * S::STEP_BYTES);
    if (ELEM || i < mine) {
      opa.load_direct(at, 0, k0);
      opb.load_direct(at + S::A_BYTES, 0, k0);
    } else {
      opa.load_direct_edge(ring + slot * S::STEP_BYTES, at, lane, 0, k0);
      opb.load_direct_edge(ring + slot * S::STEP_BYTES + S::A_BYTES, at + S::A_BYTES, lane, 0, k0);
    }
  };
#pragma unroll 1
  for (int i = 0; i < (n < D ? n : D); ++i) request(i, i);

  // ---- what the end needs is requested behind them (a count of the loads above can only be waited for too long)
  TailStep<OpA, Cfg::LA> ta;
  TailStep<OpB, Cfg::LB> tb;
  if (ELEM && tail) {
    ta.request(opa, lane, whole * STEP);
    tb.request(opb, lane, whole * STEP);
  }
  PartialTiles<TO, BM, BN, NW> end;
  end.request(p, bc);

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  typename OpA::Frag fa[KS][FM];
  typename OpB::Frag fb[KS][FN];
  auto load_frags = [&](const unsigned char* step) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int i = 0; i < FM; ++i) fa[ks][i] = opa.fragment(step, lane, 0, i, ks);
#pragma unroll
      for (int j = 0; j < FN; ++j) fb[ks][j] = opb.fragment(step + S::A_BYTES, lane, 0, j, ks);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot may be filled again
  };
  auto mfmas = [&]() {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (p.relu_a) {
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[ks][i] = relu_fragment(fa[ks][i]);
      }
      if (p.relu_b) {
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[ks][j] = relu_fragment(fb[ks][j]);
      }
      // (operands swapped: the accumulator holds C transposed, four columns of a row per lane)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = mfma_op(fb[ks][j], fa[ks][i], acc[i][j]);
    }
  };
  int slot = 0;
  for (int i = 0; i < n; ++i) {
    // whole steps in flight behind step i, at most D - 1 (the last step of K may have loads of its own behind them or,
    // where all its chunks lie outside, none: it is not counted)
    const int younger = mine - 1 - i;
    if (younger >= 3 && D >= 4)
      wait_vmcnt<(D >= 4 ? 3 : 0) * LOADS>();
    else if (younger >= 2 && D >= 3)
      wait_vmcnt<(D >= 3 ? 2 : 0) * LOADS>();
    else if (younger >= 1)
      wait_vmcnt<LOADS>();
    else
      wait_vmcnt<0>();
    load_frags(ring + slot * S::STEP_BYTES);
    if (i + D < n) request(i + D, slot);
    mfmas();
    slot = slot + 1 == D ? 0 : slot + 1;
  }
  if (ELEM && tail) {
    ta.store(opa, lane, ring);
    tb.store(opb, lane, ring + S::A_BYTES);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    load_frags(ring);
    mfmas();
  }

  __syncthreads();  // (the rings are read no more, and nothing is in flight towards them)
  end.finish(p, acc, smem, wave, lane);
}

// ---- fp32 -------------------------------------------------------------------------------------------------------------------
// An fp32 matrix instruction takes one value of each operand a lane, so fragments come straight from memory into registers,
// whatever the alignment: of four values of k in a row for each lane, 16 bytes of an operand that lies along K and four times 64
// bytes to sixteen lanes of one that does not.  Sixteen wavefronts own the steps of 16 values of k in turn and meet once, at
// the end, as above.  The order of k within a step is the same for both operands and nothing else depends on it.
// Bound by the chain of one workgroup, as above, without the round trip through LDS and the barriers for each 256 values of k
// that the shared K tiles had: microseconds queued, 256^3 4.0 -> 3.45, 64x384x400 4.7 -> 3.5, 119x323x1408 9.9 -> 6.0, 181x24x928
// 6.5 -> 4.9 on 16x16 tiles, 128x1136x1029 12.1 -> 10.6 on 32x32 ones.  Two steps of a wavefront are on their way; with four 256^3
// takes 3.6, with eight 3.9 (code for steps that a short K does not have), and a long K gains nothing.
template <int BM, int BN>
struct WaveStreamF32 {
  static constexpr int NW = 16, NT = NW * 64, STEP = 16;
  static constexpr int D = 2;
  static constexpr int LDS_BYTES = NW * BM * (BN * 4 + 16);
  static_assert(LDS_BYTES <= 160 * 1024, "LDS capacity of a gfx950 compute unit");
};

template <int BM, int BN, int LA, int LB, class Params, class S = WaveStreamF32<BM, BN>>
__global__ void __launch_bounds__(S::NT) gemm_kernel_waves_f32(const Params params) {
  const GemmParams& p = whole_params<BM, BN>(params);
  constexpr int NW = S::NW, STEP = S::STEP, D = S::D, FM = BM / 16, FN = BN / 16;
  __shared__ __attribute__((aligned(16))) unsigned char smem[S::LDS_BYTES];
  const int lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const BlockCoords bc = block_coords<BM, BN>(p);

  struct __attribute__((packed, aligned(4))) Four {
    f32x4 v;
  };
  // this lane's first values: row (column) lane % 16 of each fragment, four values of k from 4 (lane / 16) on; rows past the
  // edge are the last one again, and feed outputs that are never stored
  const float* a0 = reinterpret_cast<const float*>(p.A) + (long long)bc.batch * p.strideA;
  const float* b0 = reinterpret_cast<const float*>(p.B) + (long long)bc.batch * p.strideB;
  const int kl = bc.k_begin + 4 * (lane / 16);
  const float *pa[FM], *pb[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int m = bc.m0 + i * 16 + lane % 16, row = m < p.M ? m : p.M - 1;
    pa[i] = LA == L_KC ? a0 + (long long)row * p.lda + kl : a0 + (long long)kl * p.lda + row;
  }
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int n = bc.n0 + j * 16 + lane % 16, row = n < p.N ? n : p.N - 1;
    pb[j] = LB == L_KC ? b0 + (long long)row * p.ldb + kl : b0 + (long long)kl * p.ldb + row;
  }
  struct Step {
    f32x4 a[FM], b[FN];
  };
  auto request = [&](Step& r, int i) {  // this wavefront's step i, which lies inside K
    const long long k = (long long)(wave + i * NW) * STEP;
#pragma unroll
    for (int m = 0; m < FM; ++m) {
      if constexpr (LA == L_KC) {
        r.a[m] = reinterpret_cast<const Four*>(pa[m] + k)->v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) r.a[m][e] = pa[m][(k + e) * p.lda];
      }
    }
#pragma unroll
    for (int n = 0; n < FN; ++n) {
      if constexpr (LB == L_KC) {
        r.b[n] = reinterpret_cast<const Four*>(pb[n] + k)->v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) r.b[n][e] = pb[n][(k + e) * p.ldb];
      }
    }
  };
  f32x4 acc[FM][FN];
#pragma unroll
  for (int m = 0; m < FM; ++m)
#pragma unroll
    for (int n = 0; n < FN; ++n) acc[m][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  auto multiply = [&](Step& r) {
    if (p.relu_a) {
#pragma unroll
      for (int m = 0; m < FM; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) r.a[m][e] = r.a[m][e] < 0.0f ? 0.0f : r.a[m][e];
    }
    if (p.relu_b) {
#pragma unroll
      for (int n = 0; n < FN; ++n)
#pragma unroll
        for (int e = 0; e < 4; ++e) r.b[n][e] = r.b[n][e] < 0.0f ? 0.0f : r.b[n][e];
    }
    // (operands swapped: the accumulator holds C transposed, four columns of a row per lane)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int m = 0; m < FM; ++m)
#pragma unroll
        for (int n = 0; n < FN; ++n) acc[m][n] = mfma_op(r.b[n][e], r.a[m][e], acc[m][n]);
  };

  const int whole = bc.k_len > 0 ? bc.k_len / STEP : 0;
  const int mine = whole > wave ? (whole - wave + NW - 1) / NW : 0;
  const bool tail = whole * STEP < bc.k_len && wave == whole % NW;  // this wavefront multiplies what is left of K
  Step step[D];
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < mine) request(step[d], d);
  Step last;
  if (tail) {
    const int left = bc.k_len - whole * STEP - 4 * (lane / 16);  // values of k that this lane has
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = e < left;
      const long long k = in ? (long long)whole * STEP + e : 0;
      const long long back = in ? 0 : 4 * (lane / 16);  // (the first value of K, which there is)
#pragma unroll
      for (int m = 0; m < FM; ++m) {
        const float x = LA == L_KC ? pa[m][k - back] : pa[m][(k - back) * p.lda];
        last.a[m][e] = in ? x : 0.0f;
      }
#pragma unroll
      for (int n = 0; n < FN; ++n) {
        const float x = LB == L_KC ? pb[n][k - back] : pb[n][(k - back) * p.ldb];
        last.b[n][e] = in ? x : 0.0f;
      }
    }
  }
  PartialTiles<float, BM, BN, NW> end;
  end.request(p, bc);

  int i = 0;
  for (; i + 2 * D <= mine; i += D) {  // (without a branch: loads are counted)
#pragma unroll
    for (int d = 0; d < D; ++d) {
      multiply(step[d]);
      request(step[d], i + D + d);
    }
  }
#pragma unroll
  for (int d = 0; d < D; ++d) {
    if (i + d < mine) multiply(step[d]);
    if (i + D + d < mine) request(step[d], i + D + d);
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (i + D + d < mine) multiply(step[d]);
  if (tail) multiply(last);
  end.finish(p, acc, smem, wave, lane);
}

// ---- 16-bit types on element-aligned rows: A along K, B along N, tiles of 16 rows ---------------------------------------------
// Fragments come straight from memory here too: eight values of k of a row of A to a lane, and of B, whose rows follow k, eight
// values of a column (BN = 16) or of two neighbours (BN = 32, whose fragments hold the even and the odd columns).  There is no
// last step under predicates but what K leaves of a step, and no rows too short for it.  Sixteen wavefronts, two steps of 32
// on their way.
// Bound by the chain of one wavefront: memory latency per step, and the transactions of B's columns.  Where the rows of A lie
// a multiple of 4 bytes apart, 16x16 tiles take 0.92 of the time that direct loads into LDS take (67 random products of K up to
// 3072: 0.74 to 1.04; 80x45x796 4.16 -> 3.60 us; longer ones 1.02 to 1.10), 16x32 ones 0.90 up to K = 1024 (9 products; 7 longer
// ones 0.9 to 1.24).  Where the direct loads do not fit, as with N < 8, the general schedule is what is left: 0.42 to 0.79 of its
// time up to K = 3072 (23 products; 14x7x1264 7.8 -> 3.6 us) on any rows, 0.33 to 0.49 beyond on even ones (5x5x3768 15.5 -> 5.1),
// but 1.04 to 1.25 beyond on odd ones, where a load of 16 bytes into registers is broken up.  The fewer columns, the less the
// general schedule has to do, and the earlier that is: on odd rows 1.02 to 1.09 for two columns at K = 1281 to 1409 and 1.33 at 2945
// (300x2x2945 9.2 and 12.3 us), 0.92 to 1.03 for three up to 1793 and 1.19 at 2945, 0.82 to 1.01 for four.  Left to the loads
// into LDS: odd rows of A (0.88 to 1.58), operands that both lie along K (the same), and whole chunks, whose lines they share better (2 to 8 %).
template <int BM, int BN>
struct WaveDirect {
  static constexpr int NW = 16, NT = NW * 64, STEP = 32, D = 2;
  static constexpr int LDS_BYTES = NW * BM * (BN * 4 + 16);
  static constexpr int MAX_K = BN == 16 ? 3072 : 1024;
  static_assert(BM == 16 && (BN == 16 || BN == 32), "measured on these");
};

template <typename T, typename TO, int BM, int BN, class Params, class S = WaveDirect<BM, BN>>
__global__ void __launch_bounds__(S::NT) gemm_kernel_waves_direct(const Params params) {
  const GemmParams& p = whole_params<BM, BN>(params);
  using Frag = typename FragT<T>::type;
  constexpr int NW = S::NW, STEP = S::STEP, D = S::D, FN = BN / 16;
  constexpr bool PAIRS = FN == 2;
  __shared__ __attribute__((aligned(16))) unsigned char smem[S::LDS_BYTES];
  const int lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const BlockCoords bc = block_coords<BM, BN>(p);

  struct __attribute__((packed, aligned(2))) Eight {
    u32x4 v;
  };
  struct __attribute__((packed, aligned(2))) Two {
    unsigned v;
  };
  // this lane's first values: row lane % 16 of A, column (pair) lane % 16 of B, eight values of k from 8 (lane / 16) on; what lies
  // past an edge is the last row or column again, and feeds outputs that are never stored
  const int kl = bc.k_begin + 8 * (lane / 16);
  const int m = bc.m0 + lane % 16, n = bc.n0 + (PAIRS ? 2 : 1) * (lane % 16);
  const T* pa = reinterpret_cast<const T*>(p.A) + (long long)bc.batch * p.strideA + (long long)(m < p.M ? m : p.M - 1) * p.lda + kl;
  const T* pb = reinterpret_cast<const T*>(p.B) + (long long)bc.batch * p.strideB + (long long)kl * p.ldb;
  int down = 0;  // bits: the last column, without a neighbour, is read as the second of a pair
  if constexpr (PAIRS) {
    pb += n < p.N - 1 ? n : p.N - 2;
    down = n == p.N - 1 ? 16 : 0;
  } else {
    pb += n < p.N ? n : p.N - 1;
  }
  struct Step {
    u32x4 a;
    u32x4 b[FN];  // (pairs: the eight loads as they come)
  };
  auto request = [&](Step& r, int i) {  // this wavefront's step i, which lies inside K
    const long long k = (long long)(wave + i * NW) * STEP;
    r.a = reinterpret_cast<const Eight*>(pa + k)->v;
    if constexpr (PAIRS) {
#pragma unroll
      for (int e = 0; e < 8; ++e) r.b[e / 4][e % 4] = reinterpret_cast<const Two*>(pb + (k + e) * p.ldb)->v;
    } else {
      T t[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) t[e] = pb[(k + e) * p.ldb];
      r.b[0] = __builtin_bit_cast(u32x4, t);
    }
  };
  f32x4 acc[1][FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) acc[0][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  auto multiply = [&](const Step& r) {
    Frag fa = __builtin_bit_cast(Frag, r.a), fb[FN];
    if constexpr (PAIRS) {
      u32x4 even, odd;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned x = r.b[i / 2][2 * (i % 2)], y = r.b[i / 2][2 * (i % 2) + 1];
        odd[i] = __builtin_amdgcn_perm(y, x, 0x07060302u);
        even[i] = __builtin_amdgcn_perm(y >> down, x >> down, 0x05040100u);
      }
      fb[0] = __builtin_bit_cast(Frag, even);
      fb[1] = __builtin_bit_cast(Frag, odd);
    } else {
      fb[0] = __builtin_bit_cast(Frag, r.b[0]);
    }
    if (p.relu_a) fa = relu_fragment(fa);
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      if (p.relu_b) fb[j] = relu_fragment(fb[j]);
      acc[0][j] = mfma_op(fb[j], fa, acc[0][j]);  // (operands swapped, as above)
    }
  };

  const int whole = bc.k_len > 0 ? bc.k_len / STEP : 0;
  const int mine = whole > wave ? (whole - wave + NW - 1) / NW : 0;
  const bool tail = whole * STEP < bc.k_len && wave == whole % NW;  // this wavefront multiplies what is left of K
  Step step[D];
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < mine) request(step[d], d);
  Step last;
  if (tail) {
    const int left = bc.k_len - whole * STEP - 8 * (lane / 16);  // values of k that this lane has
    T ta[8];
    unsigned tb[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool in = e < left;
      // (outside: the first value of K, which there is, as a zero)
      const long long k = in ? (long long)whole * STEP + e : -8LL * (lane / 16);
      const T x = pa[k];
      ta[e] = in ? x : (T)0.0f;
      unsigned y;
      if constexpr (PAIRS)
        y = reinterpret_cast<const Two*>(pb + k * p.ldb)->v;
      else
        y = __builtin_bit_cast(unsigned short, pb[k * p.ldb]);
      tb[e] = in ? y : 0u;
    }
    last.a = __builtin_bit_cast(u32x4, ta);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (PAIRS)
        last.b[e / 4][e % 4] = tb[e];
      else if (e % 2 == 0)
        last.b[0][e / 2] = tb[e] | tb[e + 1] << 16;
    }
  }
  PartialTiles<TO, BM, BN, NW> end;
  end.request(p, bc);

  int i = 0;
  for (; i + 2 * D <= mine; i += D) {  // (without a branch: loads are counted)
#pragma unroll
    for (int d = 0; d < D; ++d) {
      multiply(step[d]);
      request(step[d], i + D + d);
    }
  }
#pragma unroll
  for (int d = 0; d < D; ++d) {
    if (i + d < mine) multiply(step[d]);
    if (i + D + d < mine) request(step[d], i + D + d);
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (i + D + d < mine) multiply(step[d]);
  if (tail) multiply(last);
  end.template finish<PAIRS>(p, acc, smem, wave, lane);
}

}  // namespace hidet

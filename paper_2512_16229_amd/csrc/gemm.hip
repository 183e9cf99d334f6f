// Weight-streaming bf16 GEMM for the skinny row counts of the verify step
// (M = branches x block rows, at most 2048) with fused epilogues:
//   EPI_QKV    bias + rotate-half RoPE on q/k, q -> attention input, k/v -> the
//              branch K/V staging (the Pre-Write of Sec. 3.4); always in the
//              fix-up kernel, where a thread sees both RoPE halves of a column
//   EPI_RESID  residual add into the fp32 residual stream (O-proj, down-proj)
//   EPI_SWIGLU silu(gate) * up -> packed bf16 operand of the down projection
//   EPI_LMHEAD per (row, column tile) softmax statistics: max, argmax, sum of
//              exp (the logits never reach memory)
//
// Work decomposition. The weight is a sequence of 16-column blocks; a column
// tile is NB consecutive blocks. A workgroup (4 wavefronts) covers one row tile
// (below), so each weight byte crosses HBM once per row tile, and one (column
// tile, k-split): with Q quads of k-chunks, split s owns [s Q / S, (s + 1) Q / S).
// The tile width NB and the split count S are chosen per GEMM on the host
// (plan.h):
//   S == 1  whole K in one workgroup, epilogue in place (no partial sums);
//   S  > 1  fp32 partial sums, added in split order (deterministic): for the
//           residual projections by the RMSNorm kernel that follows them, for
//           QKV by gemm_fixup_kernel, which also runs the QKV epilogue (QKV
//           always takes this path).
//
// What bounds it: the memory stream (weights from HBM, activations from L2).
// Without its MFMAs the same kernel takes the same time up to 128 rows (gate/up of
// the Dream-7B shape, 272 MB, at 32 rows: 42.3 us a workgroup, 6.4 TB/s; with
// a tile of 256 rows whatever the call's, 60 us a launch) and 0.90 to 0.97 of it in
// the short projections of 256 and 512 rows; without its loads 0.6 to 0.76. In
// gate/up and the LM head at 256 rows and more the card lowers the core clock from
// 2.4 to 1.9-2.1 GHz, which neither half does alone (gate/up at 256 rows 59 us,
// memory alone 54.5, MFMAs alone 41).
//
// Row tiles. A workgroup's tile is 64 MB rows (wavefront w: row blocks w MB ..
// w MB + MB - 1), MB = 1 .. 4 the fewest that cover the call's rows in
// ceil(rows / 256) tiles: the activation chunk a workgroup pulls per iteration
// and its MFMAs shrink with it, the weight stream stays.
//
// Pipeline. One iteration j is a 64-wide k-chunk of one tile. Its NB x 2 KiB of
// weights go global -> LDS directly (global_load_lds, no registers) into slot
// j % RING of a ring, and each wavefront's 2 MB activation fragments
// (L2-resident) into register set j % 4. Iteration j issues the activation
// loads of iteration j + 3 and the weight copies of iteration j + RING - 1. K
// is padded to a multiple of 256, so a tile always spans a multiple of 4
// iterations and the loop is unrolled by 4: no register set is ever rotated.
// Vector memory operations complete in issue order, so one vmcnt wait per
// iteration on the number of operations issued since says that the activations
// of j and the weights of j and j + 1 have landed; after the workgroup barrier
// that follows they have for every wavefront, so the weight fragments are read
// from LDS ahead of their MFMAs across the iteration boundary.
#include "common.h"
#include "kernels.h"

#include <math.h>

namespace {

constexpr int GEMM_THREADS = 256;

// Cache policy of the weight copies, by what the forward measured (us per
// launch at the Dream-7B shapes, default -> nontemporal): nontemporal where the
// stream is long or little else is read (gate/up 64.0 -> 60.2, LM head 257 -> 248
// at 256 rows; every projection at 128 rows and fewer), the default for the
// short projections of the larger row tiles (down 42.8 -> 45.4, O 18.0 -> 19.8).
constexpr bool gemm_nt(int epi, int mb) {
  return epi == EPI_SWIGLU || epi == EPI_LMHEAD || mb <= 2;
}
// wavefronts per SIMD the registers are cut for: two workgroups fit a CU's LDS
// with the narrow tile, and its registers with few row blocks
constexpr int gemm_waves(int nb, int mb) { return nb == 4 && mb <= 2 ? 2 : 1; }

template <int EPI, int NB, int MB>
struct GemmSmem {
  static constexpr int CHUNK = NB * 2048;  // bytes of weights per iteration
  static constexpr int RING = 6;
  static constexpr int BYTES = RING * CHUNK;
  static_assert(BYTES <= 160 * 1024, "LDS of one CU");
  static_assert(EPI != EPI_LMHEAD || 4 * 16 * MB * 16 * 12 <= RING * CHUNK, "reduction area fits");
};

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N <= 63, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Asynchronous global -> LDS copy of 16 bytes per lane (global_load_lds_dwordx4):
// lane l copies base + voff(l) to bytes [16 l, 16 l + 16) of the 1 KiB LDS block
// at lds_addr (wave-uniform, passed in M0). base is wave-uniform (SGPRs), so
// the only per-lane address is the constant voff = 16 lane. The compiler does
// not track the copy: completion is awaited with an explicit vmcnt wait
// before the workgroup barrier. NT selects the nontemporal (streaming) cache
// policy (gemm_nt).
__device__ __forceinline__ const void* uniform_ptr(const void* p) {
  // the "s" constraint alone does not keep a value the compiler thinks may
  // diverge out of VGPRs: make the scalar copy explicit
  const uint64_t u = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (const void*)(((uint64_t)hi << 32) | lo);
}
template <bool NT>
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t voff, uint32_t lds_addr) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 ::"s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(uniform_ptr(base))
                 : "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                 ::"s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(uniform_ptr(base))
                 : "memory");
}

// One activation fragment at a wave-uniform base + OFF -> registers.
// Issued as inline assembly so that, like the LDS copies, the compiler does not
// track them: its own waits would count only the loads it knows of and so
// stall on younger loads. Nothing reads the registers before the explicit
// vmcnt wait of the iteration that uses them; pin_landed() then hands them to
// the compiler.
template <int OFF>
__device__ __forceinline__ void load_frag(u32x4& d, const void* base, uint32_t voff) {
  asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3"
               : "=&v"(d)
               : "v"(voff), "s"(uniform_ptr(base)), "n"(OFF)
               : "memory");
}
__device__ __forceinline__ void pin_landed(u32x4& v) { asm volatile("" : "+v"(v)); }
// After the loop the last iterations' loads (repeats of the last chunk) are
// still in flight into the activation registers: wait for them, and keep the
// registers alive until then so that nothing else is placed in them earlier.
#define GEMM_DRAIN()                                                                     \
  {                                                                                      \
    wait_vmcnt<0>();                                                                     \
    _Pragma("unroll") for (int i_ = 0; i_ < 2 * MB; ++i_) {                              \
      pin_landed(a0[i_]);                                                                \
      pin_landed(a1[i_]);                                                                \
      pin_landed(a2[i_]);                                                                \
      pin_landed(a3[i_]);                                                                \
    }                                                                                    \
  }

// c += a^T b on a 16x16x32 bf16 tile, accumulating in place in AGPRs. Written as
// inline assembly with a tied operand: with the builtin the register allocator
// renames accumulators between the unrolled iterations and then copies them
// back at the loop edge. The compiler does not see these as MFMAs, so the
// hazard wait states are explicit: mfma_settle() before accumulators are read
// or rewritten by other instructions, and after they are zeroed.
__device__ __forceinline__ void mfma_acc(f32x4& c, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// FP8 (E4M3 x E4M3) form: one 16x16x128 MFMA over 32 bytes per lane of each
// operand, both operands in the default E4M3 format, unscaled (the real scales
// are applied in the epilogue; the block-scaled form with unit scales measured
// 0.3 % slower over the FP8 step). A lane's byte b of A and byte b of B meet in
// the same product, so any placement of K inside the 32 bytes works as long as
// A and W use the same.
__device__ __forceinline__ void mfma_acc_f8(f32x4& c, const u32x8& a, const u32x8& b) {
  asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ u32x8 cat8(const u32x4& lo, const u32x4& hi) {
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ void mfma_settle() {
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
}

// ------------------------------------------------------------------ epilogues
// acc[mb][nb][j]: row row0 + 16 mb + 4 g + j, column 16 (tile NB + nb) + c16
// of this wavefront (g = lane / 16, c16 = lane % 16); the SwiGLU GEMM holds
// the transposed tile (see swiglu_epilogue).

// FP8: the accumulated products times the row's and the column's scales
// (acc[mb][nb][j]: row row0 + 16 mb + 4 g + j, packed column 16 (tile NB + nb) + c16)
template <int NB, int MB>
__device__ __forceinline__ void f8_scale(const GemmArgs& a, f32x4 (&acc)[MB][NB], int tile,
                                         int row0, int lane) {
  const int g = lane >> 4, c16 = lane & 15;
  float swc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) swc[nb] = a.sw[(tile * NB + nb) * 16 + c16];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float sr = a.sa[row0 + mb * 16 + g * 4 + j];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[mb][nb][j] = acc[mb][nb][j] * sr * swc[nb];
    }
}

// One split: the residual add in place. A row block's residual values are all
// loaded (clamped, no load under a branch) before the first is used: a load per
// value under its row's test took a memory round trip each (the tiny model's
// output projection 7.4 us, 4 iterations of it).
template <int NB, int MB>
__device__ __forceinline__ void resid_epilogue(const GemmArgs& a, f32x4 (&acc)[MB][NB], int tile,
                                               int row0, int lane) {
  const int g = lane >> 4, c16 = lane & 15;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    float x[4][NB];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = row0 + mb * 16 + g * 4 + j;
      const float* xr = a.x + (int64_t)(r < a.M ? r : a.M - 1) * a.N;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int n = (tile * NB + nb) * 16 + c16;
        x[j][nb] = xr[n < a.N ? n : a.N - 1];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = row0 + mb * 16 + g * 4 + j;
      float* xr = a.x + (int64_t)r * a.N;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int n = (tile * NB + nb) * 16 + c16;
        if (r < a.M && n < a.N) xr[n] = x[j][nb] + acc[mb][nb][j];
      }
    }
  }
}

// gate / up blocks alternate (block 2p: gate columns 16p.., block 2p + 1: up);
// output block p of the tile -> columns 16 (tile NB / 2 + p) of the packed
// down-projection operand. The SwiGLU GEMM accumulates the transposed tile
// (weights as the MFMA's first operand), so acc[mb][nb][j] holds row
// row0 + 16 mb + c16, column 16 (tile NB + nb) + 4 g + j: a lane's four
// outputs of a block are four consecutive columns of one row. The packed
// operand keeps 8 consecutive columns of a row in one 16-byte lane slot, so
// lanes l and l ^ 16 (column groups 4g and 4(g ^ 1) of the same row) trade
// halves with one permlane swap per dword: afterwards the even lane holds the
// slot of row block mb, the odd lane the slot of row block mb + 1, and each
// writes 16 bytes.
template <int NB, int MB, bool F8>
__device__ __forceinline__ void swiglu_epilogue(const GemmArgs& a, f32x4 (&acc)[MB][NB], int tile,
                                                int row0, int lane) {
  constexpr int PAIRS = NB / 2;
  const int g = lane >> 4, c16 = lane & 15;
  const int Nout = a.N >> 1;
  float mxr[MB] = {};  // FP8: largest |output| of each row block's row
  auto swiglu4 = [&](int mb, int p, uint32_t (&hv)[2]) {
    // FP8: scales of the row (this lane's) and of the gate / up columns
    const float sr = F8 ? a.sa[row0 + mb * 16 + c16] : 1.f;
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      float h2[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int j = 2 * jj + u;
        float gt = acc[mb][2 * p][j], up = acc[mb][2 * p + 1][j];
        if constexpr (F8) {
          gt = gt * sr * a.sw[(tile * NB + 2 * p) * 16 + 4 * g + j];
          up = up * sr * a.sw[(tile * NB + 2 * p + 1) * 16 + 4 * g + j];
        }
        // silu(g) = g / (1 + e^-g) with the hardware exp2 and reciprocal (about
        // 1 ulp each, far below the bf16 rounding of the result)
        const float ex = __builtin_amdgcn_exp2f(-gt * 1.4426950408889634f);
        h2[u] = gt * __builtin_amdgcn_rcpf(1.0f + ex) * up;
      }
      hv[jj] = (uint32_t)f2bf_bits(h2[0]) | ((uint32_t)f2bf_bits(h2[1]) << 16);
      if constexpr (F8)
        if ((tile * PAIRS + p) * 16 < Nout)  // columns past the last block: not stored, not counted
          mxr[mb] = fmaxf(mxr[mb], fmaxf(fabsf(bf2f_bits(hv[jj] & 0xffffu)), fabsf(bf2f_bits(hv[jj] >> 16))));
    }
  };
#pragma unroll
  for (int mp = 0; mp < MB / 2; ++mp) {
    const int r = row0 + (2 * mp + (g & 1)) * 16 + c16;
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
      uint32_t h0[2], h1[2];
      swiglu4(2 * mp, p, h0);
      swiglu4(2 * mp + 1, p, h1);
      const auto w0 = __builtin_amdgcn_permlane16_swap(h0[0], h1[0], false, false);
      const auto w1 = __builtin_amdgcn_permlane16_swap(h0[1], h1[1], false, false);
      const int col = (tile * PAIRS + p) * 16 + (g >> 1) * 8;
      if (r < a.M && col < Nout)
        *(uint4*)(a.a_out + packA_off(r, col, a.Mp)) = make_uint4(w0[0], w1[0], w0[1], w1[1]);
    }
  }
  if constexpr (MB & 1) {
    // the last row block of an odd count has no partner: each lane writes its
    // four columns (8 bytes, half a slot)
    const int r = row0 + (MB - 1) * 16 + c16;
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
      uint32_t h0[2];
      swiglu4(MB - 1, p, h0);
      const int col = (tile * PAIRS + p) * 16 + 4 * g;
      if (r < a.M && col < Nout)
        *(uint2*)(a.a_out + packA_off(r, col, a.Mp)) = make_uint2(h0[0], h0[1]);
    }
  }
  if constexpr (F8) {
    // the row maxima of this tile's outputs (the stored bf16 values) into the
    // per-row maximum over all tiles: the lanes c16 + 16 g hold the same row;
    // an unsigned maximum of the bits orders non-negative floats exactly
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      float m = fmaxf(mxr[mb], __shfl_xor(mxr[mb], 16));
      m = fmaxf(m, __shfl_xor(m, 32));
      const int r = row0 + mb * 16 + c16;
      if (g == 0 && r < a.M) atomicMax(a.rowmax + r, __float_as_uint(m));
    }
  }
}

// per-row (max, argmax, sum exp(l - max)) over this tile's valid columns
// (column < vocab, column != mask token) -> pm / ps / pi [row][tile]. Each lane
// first reduces its NB columns of each of its 16 rows; the 16 lane partials of
// a row then meet in LDS (red: this wavefront's 16 MB x 16 x 3 words) and one lane
// per row merges them in column order (ties: lowest column); a row's columns are
// stored xor'd with the row, so that the lanes read 64 banks, not 4.
template <int NB, int MB>
__device__ __forceinline__ void lm_epilogue(const GemmArgs& a, f32x4 (&acc)[MB][NB], int tile,
                                            int row0, int lane, float* red) {
  constexpr float LOG2E = 1.4426950408889634f;
  const int g = lane >> 4, c16 = lane & 15;
  float* rm = red;
  constexpr int ROWS = 16 * MB;
  float* rs = red + ROWS * 16;
  int* ri = (int*)(red + 2 * ROWS * 16);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float m = -INFINITY;
      int mi = 0x7fffffff;
      float v[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int col = (tile * NB + nb) * 16 + c16;
        v[nb] = (col < a.vocab && col != a.mask_id) ? acc[mb][nb][j] : -INFINITY;
        mi = v[nb] > m ? col : mi;  // strict: the lowest column of equal maxima
        m = fmaxf(m, v[nb]);
      }
      float s = 0.f;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) s += __builtin_amdgcn_exp2f((v[nb] - m) * LOG2E);
      if (m == -INFINITY) s = 0.f;
      const int row = mb * 16 + g * 4 + j;
      const int o = row * 16 + (c16 ^ (row & 15));
      rm[o] = m;
      rs[o] = s;
      ri[o] = mi;
    }
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wavefront's LDS writes done
  __builtin_amdgcn_wave_barrier();
  float M = -INFINITY, S = 0.f;
  int I = 0x7fffffff;
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const int o = (lane < ROWS ? lane : 0) * 16 + (c ^ (lane & 15));
    const float mc = rm[o], sc = rs[o];
    const int ic = ri[o];
    if (mc > M) {
      S = S * __builtin_amdgcn_exp2f((M - mc) * LOG2E) + sc;
      M = mc;
      I = ic;
    } else if (mc == M) {
      S += sc;
      I = ic < I ? ic : I;
    } else {
      S += sc * __builtin_amdgcn_exp2f((mc - M) * LOG2E);
    }
  }
  const int r = row0 + lane;
  if (lane < ROWS && r < a.M) {
    const int64_t o = (int64_t)r * a.tiles + tile;
    a.pm[o] = M;
    a.ps[o] = M == -INFINITY ? 0.f : S;
    a.pi[o] = I;
  }
}

// ------------------------------------------------------------------ main loop
// Loads of one iteration: 2 MB activation fragments into register set `set`
// (two groups of MB, k-halves 0 and 1) and the NB x 2 KiB weight chunk into
// ring slot `slot` (NB / 2 copies of 1 KiB per wavefront). Weight layout
// [KC][blocks][2][64 lanes][8]: the chunk of (tile, kc) is one contiguous run,
// and the workgroups, which advance in step, read neighbouring runs at a time.
// The activation and the weight addresses advance by one k-chunk per issued
// iteration, from kc0 to the end of the range and then from its start
// (rotation, GemmArgs::rot); after the last of the range's iterations the last
// chunk is issued again (an L2 hit), which keeps every wait count constant and
// the loop branch-free.
#define GEMM_ISSUE_A(set, i) /* fragment i < 2 MB: row block i % MB, k-half i / MB */    \
  switch ((i) % MB) {                                                                    \
    case 0: load_frag<0>(set[i], a_next + ((i) / MB) * a_half, voff); break;             \
    case 1: load_frag<1024>(set[i], a_next + ((i) / MB) * a_half, voff); break;          \
    case 2: load_frag<2048>(set[i], a_next + ((i) / MB) * a_half, voff); break;          \
    case 3: load_frag<3072>(set[i], a_next + ((i) / MB) * a_half, voff); break;          \
  }
#define GEMM_ISSUE_W(r, slot)                                                            \
  lds_dma16<NT>(w_next + (r) * 4096, voff,                                               \
                lds_wave + (uint32_t)(slot) * (uint32_t)SM::CHUNK + (uint32_t)(r) * 4096u)
#define GEMM_ADVANCE(next, step, back, li, lk)                                           \
  {                                                                                      \
    const bool more_ = li + 1 < n_it, wrap_ = lk + 1 == kc_end;                          \
    const int64_t d_ = wrap_ ? -back : step;                                             \
    next += more_ ? d_ : 0;                                                              \
    lk = more_ ? (wrap_ ? kc_beg : lk + 1) : lk;                                         \
    ++li;                                                                                \
  }
#define GEMM_ISSUE_A_ALL(set)                                                            \
  {                                                                                      \
    _Pragma("unroll") for (int i_ = 0; i_ < 2 * MB; ++i_) GEMM_ISSUE_A(set, i_);         \
    GEMM_ADVANCE(a_next, a_kstep, a_back, lia, lka);                                             \
  }
#define GEMM_ISSUE_W_ALL(slot)                                                           \
  {                                                                                      \
    _Pragma("unroll") for (int r_ = 0; r_ < NB / 2; ++r_) GEMM_ISSUE_W(r_, slot);        \
    GEMM_ADVANCE(w_next, w_kstep, w_back, liw, lkw);                                             \
  }

// Iteration j on register set `cur` (j % 4), issuing the activations of j + 3
// into `nxt` ((j + 3) % 4, last read by iteration j - 1) and the weights of
// j + RING - 1 into the slot that iteration j - 1 read (every wavefront is past
// it after this barrier). Its 2 NB weight fragments f are read from LDS BPF
// ahead of their MFMAs into bf[f % BPF], the last BPF reads being the next
// iteration's first fragments. The loads are spread evenly over the MFMA stream (a wavefront
// that waits for a full memory queue issues no MFMA);
// scheduling barriers keep the order. FP8: a fragment covers 64 values of K (16
// per lane) and they are read in (block, half) order, so that both halves of a
// block are in registers together; each block takes one 16x16x128 MFMA per row
// block. In bf16 the order is (half, block).
#define GEMM_LDS_FRAG(slot, f)                                                           \
  ((const u32x4*)(smem + (slot) * SM::CHUNK))[(F8 ? (f) : ((f) % NB) * 2 + (f) / NB) * 64 + lane]
#define GEMM_ITER(cur, nxt)                                                              \
  {                                                                                      \
    wait_vmcnt<WAIT>();                                                                  \
    lds_barrier();                                                                       \
    _Pragma("unroll") for (int i_ = 0; i_ < 2 * MB; ++i_) pin_landed(cur[i_]);           \
    const int ns_ = cs + 1 == SM::RING ? 0 : cs + 1;                                     \
    const int is_ = cs == 0 ? SM::RING - 1 : cs - 1;                                     \
    __builtin_amdgcn_sched_barrier(0);                                                   \
    _Pragma("unroll") for (int f_ = 0; f_ < 2 * NB; ++f_) {                              \
      if constexpr (F8) {                                                                \
        if (f_ & 1) {                                                                    \
          const u32x8 b8_ = cat8(bf[(f_ - 1) % BPF], bf[f_ % BPF]);                      \
          _Pragma("unroll") for (int mb_ = 0; mb_ < MB; ++mb_) {                         \
            const u32x8 a8_ = cat8(cur[mb_], cur[MB + mb_]);                             \
            if constexpr (EPI == EPI_SWIGLU)                                             \
              mfma_acc_f8(acc[mb_][f_ >> 1], b8_, a8_);                                  \
            else                                                                         \
              mfma_acc_f8(acc[mb_][f_ >> 1], a8_, b8_);                                  \
          }                                                                              \
          _Pragma("unroll") for (int u_ = f_ - 1; u_ <= f_; ++u_)                        \
            bf[u_ % BPF] = GEMM_LDS_FRAG(u_ + BPF < 2 * NB ? cs : ns_, (u_ + BPF) % (2 * NB)); \
        }                                                                                \
      } else {                                                                           \
        _Pragma("unroll") for (int mb_ = 0; mb_ < MB; ++mb_)                             \
          if constexpr (EPI == EPI_SWIGLU) /* transposed tile: lanes hold output rows */ \
            mfma_acc(acc[mb_][f_ % NB], bf[f_ % BPF], cur[(f_ / NB) * MB + mb_]);        \
          else                                                                           \
            mfma_acc(acc[mb_][f_ % NB], cur[(f_ / NB) * MB + mb_], bf[f_ % BPF]);        \
        bf[f_ % BPF] = GEMM_LDS_FRAG(f_ + BPF < 2 * NB ? cs : ns_, (f_ + BPF) % (2 * NB)); \
      }                                                                                  \
      _Pragma("unroll") for (int o_ = 0; o_ < OPS; ++o_)                                 \
        if (o_ * 2 * NB / OPS == f_) {                                                   \
          if (o_ < 2 * MB) {                                                             \
            GEMM_ISSUE_A(nxt, o_);                                                       \
            if (o_ == 2 * MB - 1) GEMM_ADVANCE(a_next, a_kstep, a_back, lia, lka);       \
          } else {                                                                       \
            GEMM_ISSUE_W(o_ - 2 * MB, is_);                                              \
            if (o_ == OPS - 1) GEMM_ADVANCE(w_next, w_kstep, w_back, liw, lkw);          \
          }                                                                              \
        }                                                                                \
      __builtin_amdgcn_sched_barrier(0);                                                 \
    }                                                                                    \
    cs = ns_;                                                                            \
  }

template <int EPI, int NB, int MB, bool F8>
__global__ __launch_bounds__(GEMM_THREADS, 1) __attribute__((amdgpu_waves_per_eu(gemm_waves(NB, MB), gemm_waves(NB, MB)))) void gemm_kernel(GemmArgs a) {
  using SM = GemmSmem<EPI, NB, MB>;
  // FP8: the epilogues of RESID and LMHEAD take scaled sums (f8_scale), SWIGLU
  // scales inside its epilogue, QKV in the fix-up (its partial sums are raw)
  constexpr int OPS = 2 * MB + NB / 2;  // vector memory operations per wavefront per iteration
  // operations in flight at the top of iteration j: those of the last two
  // iterations (activations of j + 1 and j + 2, weights of j + 3 and j + 4)
  constexpr int WAIT = 2 * OPS;
  constexpr int BPF = MB >= 3 ? 4 : NB == 10 ? 10 : 8;  // fragments read ahead (LDS latency)
  constexpr bool NT = gemm_nt(EPI, MB);
  static_assert(NB % 2 == 0 && NB <= GEMM_MAX_NB && SM::RING == 6, "tile");
  static_assert(WAIT <= 63 && 2 * NB % BPF == 0, "pipeline");
  __shared__ __attribute__((aligned(1024))) char smem[SM::BYTES];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t sW_base = (uint32_t)(uintptr_t)smem;

  // Hardware places workgroup b on XCD b % 8; the remap gives each XCD a
  // contiguous range of q (XCD x: grid / 8 workgroups, one more when x <
  // grid % 8), so the row tiles of one column workgroup (adjacent q) share an
  // L2 and read each weight chunk from HBM once.
  const int b = blockIdx.x, grid = gridDim.x;
  const int xcd = b & 7, g8 = grid >> 3, g8r = grid & 7;
  const int q = xcd * g8 + (xcd < g8r ? xcd : g8r) + (b >> 3);
  const int MT = a.mtiles;
  const int mt = q % MT, c = q / MT;
  const int KC = a.KC, QT = KC >> 2;
  // workgroup c of a row tile: k-split c / T, column tile c % T. Split-major, so
  // that the workgroups of one XCD (consecutive q) share a k-range and with it
  // the slice of the activation operand they stream: it stays in that XCD's
  // L2 instead of being fetched once per column tile.
  const int split = c / a.tiles;
  const int t_lo = c % a.tiles;
  const int kc_beg = 4 * (split * QT / a.splits);
  const int kc_end = 4 * ((split + 1) * QT / a.splits);
  if (t_lo >= a.tiles || kc_beg >= kc_end) return;
  const int nq = (kc_end - kc_beg) >> 2;  // quads of iterations per tile
  const int RB = a.Mp >> 4;
  const int rb0 = (mt * 4 + wv) * MB;  // first 16-row block of this wavefront
  const int row0 = rb0 * 16;           // first row of this wavefront
  const uint32_t voff = (uint32_t)lane * 16u;
  // activation fragment (kb, rb) at A + ((kb RB) + rb) KiB: k-chunk kc, half h
  // of this wavefront's first row block -> a_next + h a_half
  const int64_t a_half = (int64_t)RB * 1024, a_kstep = 2 * a_half;
  const int n_it = kc_end - kc_beg;  // iterations of this workgroup
  const int kc0 = kc_beg + (a.rot ? 4 * (t_lo % nq) : 0);  // first k-chunk
  const char* a_next = (const char*)a.A + ((int64_t)2 * kc0 * RB + rb0) * 1024;
  // weight chunk (tile, kc) at W + (kc blocks + tile NB) 2 KiB; its 1 KiB unit u
  // (block u / 2, k-half u % 2) at + u KiB; wavefront wv copies units 4 r + wv
  const int64_t w_kstep = (int64_t)a.wblocks * 2048;
  const char* w_next = (const char*)a.W + kc0 * w_kstep + (int64_t)t_lo * SM::CHUNK + wv * 1024;
  const uint32_t lds_wave = sW_base + (uint32_t)wv * 1024u;
  const int64_t a_back = (n_it - 1) * a_kstep, w_back = (n_it - 1) * w_kstep;  // range end -> start
  int lka = kc0, lkw = kc0;  // k-chunk of the next iteration to issue (activations, weights)
  int lia = 0, liw = 0;      // iterations issued before it

  f32x4 acc[MB][NB];
  u32x4 a0[2 * MB], a1[2 * MB], a2[2 * MB], a3[2 * MB];
  u32x4 bf[BPF];
  GEMM_ISSUE_W_ALL(0);
  GEMM_ISSUE_W_ALL(1);
  GEMM_ISSUE_A_ALL(a0);
  GEMM_ISSUE_W_ALL(2);
  GEMM_ISSUE_A_ALL(a1);
  GEMM_ISSUE_W_ALL(3);
  GEMM_ISSUE_A_ALL(a2);
  GEMM_ISSUE_W_ALL(4);
  int cs = 0;  // ring slot of the current iteration

  {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    mfma_settle();
    // the first iteration's first fragments
    wait_vmcnt<WAIT>();
    lds_barrier();
#pragma unroll
    for (int f = 0; f < BPF; ++f) bf[f] = GEMM_LDS_FRAG(0, f);
    int qq = nq;
    do {
      GEMM_ITER(a0, a3);
      GEMM_ITER(a1, a0);
      GEMM_ITER(a2, a1);
      GEMM_ITER(a3, a2);
    } while (--qq > 0);
    GEMM_DRAIN();
    mfma_settle();
    if constexpr (F8 && (EPI == EPI_RESID || EPI == EPI_LMHEAD))
      f8_scale<NB, MB>(a, acc, t_lo, row0, lane);
    if (EPI != EPI_QKV && a.splits == 1) {
      if constexpr (EPI == EPI_LMHEAD) {
        lds_barrier();  // the ring becomes the reduction area (every copy has landed)
        lm_epilogue<NB, MB>(a, acc, t_lo, row0, lane, (float*)smem + wv * 16 * MB * 16 * 3);
      }
      if constexpr (EPI == EPI_RESID) resid_epilogue<NB, MB>(a, acc, t_lo, row0, lane);
      if constexpr (EPI == EPI_SWIGLU) swiglu_epilogue<NB, MB, F8>(a, acc, t_lo, row0, lane);
    } else if constexpr (EPI == EPI_RESID) {
      // row-major partial sums [split][Mp][N], added by the following RMSNorm
      const int g = lane >> 4, c16 = lane & 15;
      float* part = a.partials + (int64_t)split * a.Mp * a.N;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        if (row0 + mb * 16 < a.M)  // row blocks of padding alone are never read
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float* pr = part + (int64_t)(row0 + mb * 16 + g * 4 + j) * a.N;
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            const int n = (t_lo * NB + nb) * 16 + c16;
            if (n < a.N) pr[n] = acc[mb][nb][j];
          }
        }
    } else {
      const int64_t slot = ((int64_t)mt * a.tiles + t_lo) * a.splits + split;
      f32x4* part = (f32x4*)a.partials + (slot * 4 + wv) * MB * NB * 64;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) part[(mb * NB + nb) * 64 + lane] = acc[mb][nb];
    }
  }
  wait_vmcnt<0>();  // nothing may still be writing LDS when the workgroup ends
}

// QKV: sum the S partials of one f32x4 of the output (4 rows, 1 column) in
// split order and run the epilogue. A wavefront per (row block, 16-column block),
// the same indexing as gemm_kernel's partial store, so each wavefront's load is
// 1 KiB contiguous. The split count SC (1..8, QKV_MAX_SPLITS) is a constant, so
// that every load of a thread (the split sums of its column and of its rotation
// partner, the rotary rows, bias and scales) is in flight before the first add.
template <int SC>
__global__ __launch_bounds__(256) void gemm_fixup_kernel(GemmArgs a) {
  const int lane = threadIdx.x & 63;
  const int blk = blockIdx.y * 4 + (threadIdx.x >> 6);  // 16-column block
  const int NB = a.nb, MB = a.mb, lnb = 31 - __builtin_clz(NB);  // NB a power of two
  // row block blockIdx.x of row tile mt: wavefront wv, its block mb
  const int mt = blockIdx.z, wm = blockIdx.x;
  const int wv = (wm >= MB) + (wm >= 2 * MB) + (wm >= 3 * MB), mb = wm - wv * MB;
  const int g = lane >> 4, c16 = lane & 15;
  const int r0 = (mt * 4 * MB + wm) * 16 + g * 4;
  const int n = blk * 16 + c16;
  if (n >= a.N || r0 >= a.M) return;
  const int D = a.d, HD = D >> 1;
  const int qcols = a.Hq * D, kcols = a.Hkv * D;
  const int sect = n < qcols ? 0 : (n < qcols + kcols ? 1 : 2);
  const int base = sect == 0 ? 0 : (sect == 1 ? qcols : qcols + kcols);
  const int ld = __builtin_ctz(D);  // D = 64 or 128
  const int head = (n - base) >> ld, dim = (n - base) & (D - 1);
  if (sect < 2 && dim >= HD) return;  // written with its rotation partner
  const bool rot = sect < 2;
  const int n2 = rot ? n + HD : n;  // the partner column (V: the column itself, unused)
  const int64_t sstride = (int64_t)4 * MB * NB * 64;  // f32x4 between consecutive splits
  auto first = [&](int col) {
    const int t2 = (col >> 4) >> lnb, nb2 = (col >> 4) & (NB - 1);
    return (const f32x4*)a.partials +
           ((((int64_t)mt * a.tiles + t2) * a.splits * 4 + wv) * MB * NB + mb * NB + nb2) * 64 + lane;
  };
  const f32x4* p1 = first(n);
  const f32x4* p2 = first(n2);
  f32x4 v1 = p1[0], v2 = p2[0];
#pragma unroll
  for (int s = 1; s < SC; ++s) {
    v1 += p1[s * sstride];
    v2 += p2[s * sstride];
  }
  // rows r0 .. r0 + 3 (those past M are not stored; their position is some row's of a block)
  int br[4], pos[4];
  float2 cs[4];
  float sr[4];
  const int br0 = r0 / a.L, pos0 = r0 - br0 * a.L;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    // a block may be shorter than four rows
    br[j] = j == 0 ? br0 : pos[j - 1] + 1 == a.L ? br[j - 1] + 1 : br[j - 1];
    pos[j] = j == 0 ? pos0 : pos[j - 1] + 1 == a.L ? 0 : pos[j - 1] + 1;
    const int at = a.P + (!a.chain ? pos[j] : r0 + j < a.M ? r0 + j : 0);  // position of the row
    cs[j] = rot ? *(const float2*)(a.rope + ((int64_t)at * HD + dim) * 2)
                : make_float2(1.f, 0.f);
    sr[j] = a.f8 && r0 + j < a.M ? a.sa[r0 + j] : 0.f;
  }
  const float b1 = a.bias ? a.bias[n] : 0.f;
  const float b2 = (a.bias && rot) ? a.bias[n2] : 0.f;
  const float sw1 = a.f8 ? a.sw[n] : 0.f, sw2 = a.f8 && rot ? a.sw[n2] : 0.f;
  if (a.f8) {  // FP8 operands: the sums of products times the row and column scales
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v1[j] = v1[j] * sr[j] * sw1;
      if (rot) v2[j] = v2[j] * sr[j] * sw2;
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (r0 + j >= a.M) continue;
    const int i = pos[j];
    float o1 = v1[j] + b1, o2 = 0.f;
    if (rot) {
      const float x1 = o1, x2 = v2[j] + b2;
      o1 = x1 * cs[j].x - x2 * cs[j].y;
      o2 = x2 * cs[j].x + x1 * cs[j].y;
    }
    if (sect == 0) {
      uint16_t* qo = a.q_out + (((int64_t)br[j] * a.Hq + head) * a.L + i) * D;
      qo[dim] = f2bf_bits(o1);
      qo[dim + HD] = f2bf_bits(o2);
    } else {
      // K or V of this head, in the KV tile layout: position i of a region
      auto put = [&](uint16_t* st, int i) {
        if (sect == 1) {
          st[kv_k_off(i, dim, D)] = f2bf_bits(o1);
          st[kv_k_off(i, dim + HD, D)] = f2bf_bits(o2);
        } else {
          st[kv_v_off(i, dim, D)] = f2bf_bits(o1);
        }
      };
      if (a.chain)
        put((sect == 1 ? a.kcache : a.vcache) + (int64_t)head * D * a.vld, a.P + r0 + j);
      if (!a.chain || br[j] == a.stage_block)  // staging of this branch and layer
        put(a.staging + ((((int64_t)(a.chain ? 0 : br[j]) * a.layers + a.layer) * 2 + (sect - 1)) *
                             a.Hkv + head) * D * a.vlds, i);
    }
  }
}

template <int EPI, int NB, int MB, bool F8>
hipError_t launch_tile(const GemmArgs& a, hipStream_t s) {
  const int grid = a.mtiles * a.gcols;
  hipLaunchKernelGGL((gemm_kernel<EPI, NB, MB, F8>), dim3(grid), dim3(GEMM_THREADS), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_fixup(const GemmArgs& a, hipStream_t s) {
  const dim3 fg((unsigned)(4 * a.mb), (unsigned)((a.N / 16 + 3) / 4), (unsigned)a.mtiles);
  switch (a.splits) {
#define FIXUP(SC) case SC: hipLaunchKernelGGL((gemm_fixup_kernel<SC>), fg, dim3(256), 0, s, a); break
    FIXUP(1);
    FIXUP(2);
    FIXUP(3);
    FIXUP(4);
    FIXUP(5);
    FIXUP(6);
    FIXUP(7);
    FIXUP(8);
    default: return hipErrorInvalidValue;  // launch_gemm admits at most QKV_MAX_SPLITS
#undef FIXUP
  }
  return hipGetLastError();
}

template <int EPI, int NB, bool F8>
hipError_t launch_rows(const GemmArgs& a, hipStream_t s) {
  hipError_t e = hipErrorInvalidValue;
  switch (a.mb) {
    case 1: e = launch_tile<EPI, NB, 1, F8>(a, s); break;
    case 2: e = launch_tile<EPI, NB, 2, F8>(a, s); break;
    case 3: e = launch_tile<EPI, NB, 3, F8>(a, s); break;
    case 4: e = launch_tile<EPI, NB, 4, F8>(a, s); break;
  }
  if (EPI == EPI_QKV && e == hipSuccess) e = launch_fixup(a, s);
  return e;
}

template <bool F8>
hipError_t launch_epi(int epi, const GemmArgs& a, hipStream_t s) {
  switch (epi * 32 + a.nb) {
    case EPI_QKV * 32 + 4: return launch_rows<EPI_QKV, 4, F8>(a, s);
    case EPI_QKV * 32 + 8: return launch_rows<EPI_QKV, 8, F8>(a, s);
    case EPI_RESID * 32 + 4: return launch_rows<EPI_RESID, 4, F8>(a, s);
    case EPI_RESID * 32 + 8: return launch_rows<EPI_RESID, 8, F8>(a, s);
    case EPI_SWIGLU * 32 + 4: return launch_rows<EPI_SWIGLU, 4, F8>(a, s);
    case EPI_SWIGLU * 32 + 8: return launch_rows<EPI_SWIGLU, 8, F8>(a, s);
    case EPI_SWIGLU * 32 + 10: return launch_rows<EPI_SWIGLU, 10, F8>(a, s);
    case EPI_LMHEAD * 32 + 4: return launch_rows<EPI_LMHEAD, 4, F8>(a, s);
    case EPI_LMHEAD * 32 + 8: return launch_rows<EPI_LMHEAD, 8, F8>(a, s);
    case EPI_LMHEAD * 32 + 10: return launch_rows<EPI_LMHEAD, 10, F8>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_gemm(int epi, const GemmArgs& a, hipStream_t s) {
  // (epilogue, tile width) pairs the host planner may choose; splits > 1 only
  // for EPI_QKV and EPI_RESID
  if (a.splits > 1 && (epi == EPI_SWIGLU || epi == EPI_LMHEAD)) return hipErrorInvalidValue;
  if (a.KC % 4 || a.KC < 4 || a.splits < 1 || a.splits > a.KC / 4 || a.mtiles < 1 ||
      a.gcols < 1 || a.mb < 1 || a.mb > 4 || a.Mp != 64 * a.mb * a.mtiles || a.M > a.Mp)
    return hipErrorInvalidValue;
  if (a.gcols != a.tiles * a.splits || a.tiles * a.nb < a.wblocks ||
      (a.tiles - 1) * a.nb >= a.wblocks)
    return hipErrorInvalidValue;
  if (epi == EPI_QKV && a.splits > QKV_MAX_SPLITS) return hipErrorInvalidValue;
  if (a.f8) {
    if (!a.sa || !a.sw || (epi == EPI_SWIGLU && !a.rowmax)) return hipErrorInvalidValue;
    return launch_epi<true>(epi, a, s);
  }
  return launch_epi<false>(epi, a, s);
}

// Decomposition of a verify forward's GEMMs and the sizes of its working memory,
// by row count: host arithmetic without any HIP, so that a host program can check
// it over whole ranges of shapes.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "../../include/lopa.h"

enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_LMHEAD = 3 };
// most k-splits of the QKV projection (its fix-up sums them with the count as a constant)
constexpr int QKV_MAX_SPLITS = 8;

// What the plans depend on.
struct ModelShape {
  lopa_model_cfg cfg = {};
  int num_cu = 0;
  int n_qkv = 0;
  int blk_qkv = 0, blk_h = 0, blk_gu = 0, blk_lm = 0;  // packed 16-column blocks
  int fp8 = 0;         // FP8 MLP (LOPA_PRECISION_FP8_MLP and LOPA_PRECISION_FP8)
  int fp8_qkv_lm = 0;  // FP8 QKV projection and LM head too (LOPA_PRECISION_FP8)
  void set(const lopa_model_cfg& c, int precision) {
    cfg = c;
    n_qkv = (c.heads + 2 * c.kv_heads) * c.head_dim;
    blk_qkv = n_qkv / 16;
    blk_h = c.hidden / 16;
    blk_gu = 2 * c.ffn / 16;
    blk_lm = (c.vocab + 15) / 16;
    fp8 = precision == LOPA_PRECISION_FP8_MLP || precision == LOPA_PRECISION_FP8;
    fp8_qkv_lm = precision == LOPA_PRECISION_FP8;
  }
};

inline int round256(int k) { return 256 * ((k + 255) / 256); }
inline int round512(int k) { return 512 * ((k + 511) / 512); }
inline int round_up(int x, int m) { return m * ((x + m - 1) / m); }

// Row tiles of a forward of M rows: MT = ceil(M / 256) tiles of 64 mb rows each,
// mb (1..4) the smallest that covers M, so few rows stream few activations.
struct RowTiles {
  int MT, mb;
  int rows() const { return 64 * mb * MT; }
  int index() const { return (MT - 1) * 4 + mb - 1; }
};
inline RowTiles row_tiles(int M) {
  const int MT = (M + 255) / 256;
  return {MT, ((M + MT - 1) / MT + 63) / 64};
}
// rows of the packed activation buffers of a forward of up to M rows (a smaller
// forward never takes more: its tiles are as many or fewer, of 256 rows at most)
inline int padded_rows(int M) { return 256 * ((M + 255) / 256); }

// Decomposition of one GEMM (see gemm.hip): tile width nb (16-column blocks)
// and k-splits S; SwiGLU and LM head take no split (their epilogues need whole
// sums). The pair with the smallest estimated time is taken. A round of
// workgroups (one per CU) takes the longest of
//   (a) the bytes one workgroup pulls into its CU, per 64-wide k-chunk the
//       64 mb x 64 activation chunk from L2 and nb x 2 KiB of weights (61 GB/s),
//   (b) the round's weight bytes from HBM (7.2 TB/s),
//   (c) its MFMAs, 5 ns per row block and 32 x 16 weight fragment,
// plus 0.27 of the shorter of (a) and (c), which overlap in part, plus 0.9 us of
// fill and tail. Partial sums add their write (5.8 TB/s) and the read of
// the kernel that adds them (3 TB/s). The constants are fitted to the GEMM
// shapes of Dream-7B and LLaDA-8B. Against every (nb, S) timed on its own (both
// layouts, bf16 and FP8, ten row counts from 32 to 2048, the five GEMMs: 200
// choices) the plan taken is 0.4 % slower than the fastest in the mean, 12 % in
// the worst case (LLaDA-8B's output projection at 64 rows, 75 us a forward against
// 68).
// max_part: most bytes of partial sums (splits that write more are not taken;
// QKV keeps one split at least). min_nb: narrowest tile.
struct GemmPlan {
  int nb, tiles, splits;
};
inline GemmPlan plan_gemm(int epi, int nblocks, int KC, RowTiles rt, int num_cu,
                   size_t max_part = SIZE_MAX, int min_nb = 4) {
  constexpr double CU_BPUS = 61e3, HBM_BPUS = 7.2e6, PART_W_BPUS = 5.8e6, PART_R_BPUS = 3e6;
  constexpr double FRAG_US = 0.005, OVERLAP = 0.27, FILL_US = 0.9;
  const bool whole = epi == EPI_SWIGLU || epi == EPI_LMHEAD;
  const int Q = KC / 4;
  const int max_s = whole ? 1 : epi == EPI_QKV ? std::min(Q, QKV_MAX_SPLITS) : Q;
  GemmPlan best{0, 0, 0};
  double best_t = 1e300;
  for (int nb : {4, 8, 10}) {
    if (nb < min_nb || (nb == 10 && !whole)) continue;
    const int tiles = (nblocks + nb - 1) / nb;
    for (int S = 1; S <= max_s; ++S) {
      const int64_t wgs = (int64_t)rt.MT * tiles * S;
      if (S > 1 && (wgs > 8 * (int64_t)num_cu ||
                    (size_t)S * rt.rows() * tiles * nb * 16 * 4 > max_part))
        break;
      const int64_t rounds = (wgs + num_cu - 1) / num_cu;
      const double iters = 4.0 * ((Q + S - 1) / S);
      const double cu = iters * (rt.mb * 8192.0 + nb * 2048.0) / CU_BPUS;
      const double mfma = iters * rt.mb * nb * 2 * FRAG_US;
      const double hbm = (double)std::min<int64_t>(wgs, num_cu) / rt.MT * iters * nb * 2048.0 / HBM_BPUS;
      double t = (double)rounds * (FILL_US + std::max({cu, mfma, hbm}) + OVERLAP * std::min(cu, mfma));
      if (epi == EPI_QKV || S > 1) {
        const double part = (double)S * rt.rows() * nblocks * 16 * 4;
        t += part / PART_W_BPUS + part / PART_R_BPUS;
      }
      if (t < best_t) {
        best_t = t;
        best = {nb, tiles, S};
      }
    }
  }
  return best;
}
// bytes of fp32 partial sums the plan writes (QKV always goes through them;
// the residual projections store [splits][rows][N] row-major)
inline size_t plan_partial_bytes(int epi, const GemmPlan& p, RowTiles rt, int nblocks) {
  if (epi == EPI_QKV) return (size_t)rt.rows() * p.tiles * p.nb * 16 * 4 * p.splits;
  return p.splits > 1 ? (size_t)p.splits * rt.rows() * nblocks * 16 * 4 : 0;
}

// the row tiles and the plans of the five GEMMs of a verify forward
struct StepPlans {
  RowTiles rt;
  GemmPlan qkv, o, gu, down, lm;
};
inline StepPlans plan_step(const ModelShape* m, RowTiles rt, size_t max_part = SIZE_MAX, int min_nb_lm = 4) {
  const lopa_model_cfg& c = m->cfg;
  const int kch = m->fp8_qkv_lm ? round512(c.hidden) / 128 : c.hidden / 64;
  const int kco = m->fp8_qkv_lm ? round512(c.heads * c.head_dim) / 128 : c.heads * c.head_dim / 64;
  const int kcg = m->fp8 ? round512(c.hidden) / 128 : c.hidden / 64;
  const int kcd = m->fp8 ? round512(c.ffn) / 128 : round256(c.ffn) / 64;
  StepPlans p;
  p.rt = rt;
  p.qkv = plan_gemm(EPI_QKV, m->blk_qkv, kch, rt, m->num_cu, max_part);
  p.o = plan_gemm(EPI_RESID, m->blk_h, kco, rt, m->num_cu, max_part);
  p.gu = plan_gemm(EPI_SWIGLU, m->blk_gu, kcg, rt, m->num_cu);
  p.down = plan_gemm(EPI_RESID, m->blk_h, kcd, rt, m->num_cu, max_part);
  p.lm = plan_gemm(EPI_LMHEAD, m->blk_lm, kch, rt, m->num_cu, SIZE_MAX, min_nb_lm);
  return p;
}
// bytes of partial sums and LM-head (row, tile) statistics of a forward
inline size_t partial_bytes(const ModelShape* m, const StepPlans& p) {
  return std::max({(size_t)16, plan_partial_bytes(EPI_QKV, p.qkv, p.rt, m->blk_qkv),
                   plan_partial_bytes(EPI_RESID, p.o, p.rt, m->blk_h),
                   plan_partial_bytes(EPI_RESID, p.down, p.rt, m->blk_h)});
}
inline size_t lm_stats(const StepPlans& p) { return (size_t)p.rt.rows() * p.lm.tiles; }

// the plans of every row count up to max_rows, by RowTiles::index()
inline std::vector<StepPlans> all_plans(const ModelShape* m, int max_rows) {
  std::vector<StepPlans> v((size_t)(max_rows + 255) / 256 * 4, StepPlans{});
  for (int M = 1; M <= max_rows; ++M) {
    const RowTiles rt = row_tiles(M);
    StepPlans& p = v[rt.index()];
    if (p.rt.MT == 0) p = plan_step(m, rt);
  }
  return v;
}

// A forward's working memory in one piece (byte offsets, multiples of 256).
// Regions whose contents are never alive together lie on top of each other:
//   shared  the split-K partial sums and the attention's scratch, each consumed by
//           the kernel after its producer; after the last layer the LM head's
//           statistics. FP8 models keep the SwiGLU rows here too: O's partial sums
//           are added before gate/up writes them, and they are requantised (a8_dn)
//           before the down projection writes its own.
//   qbuf    the queries, read by the attention before gate/up writes the SwiGLU
//           rows: at the start of fbuf in bf16 models where it ends below fbuf's
//           padding columns (which the embedding kernel zeroes once a forward).
struct WsLayout {
  size_t x = 0, abuf = 0, fbuf = 0, qbuf = 0, shared = 0, shared_bytes = 0;
  size_t a8_gu = 0, a8_dn = 0, sa_gu = 0, sa_dn = 0, rowmax_dn = 0;  // FP8 models
  size_t stats_bytes = 0;  // one of the three LM-head statistics
  size_t total = 0;
};
// M rows; scratch: the attention's
inline WsLayout ws_layout(const ModelShape* m, const StepPlans& p, int M, size_t scratch) {
  const lopa_model_cfg& c = m->cfg;
  const size_t rows = p.rt.rows();
  WsLayout w;
  auto round = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
  auto take = [&](size_t bytes) {
    const size_t at = w.total;
    w.total += round(bytes);
    return at;
  };
  const size_t f_bytes = rows * round256(c.ffn) * 2, q_bytes = (size_t)M * c.heads * c.head_dim * 2;
  w.stats_bytes = round(lm_stats(p) * 4);
  w.shared_bytes = round(std::max({partial_bytes(m, p), scratch, 3 * w.stats_bytes}));
  w.x = take(rows * c.hidden * 4);
  w.abuf = take(rows * c.hidden * 2);
  if (m->fp8) {
    w.fbuf = w.shared = take(std::max(w.shared_bytes, f_bytes));
    w.qbuf = take(q_bytes);
    w.a8_gu = take(rows * round512(c.hidden));
    w.a8_dn = take(rows * round512(c.ffn));
    w.sa_gu = take(rows * 4);
    w.sa_dn = take(rows * 4);
    w.rowmax_dn = take(rows * 4);
  } else {
    w.shared = take(w.shared_bytes);
    w.fbuf = take(f_bytes);
    w.qbuf = q_bytes <= rows * (c.ffn / 32 * 32) * 2 ? w.fbuf : take(q_bytes);
  }
  return w;
}
// The plan of a forward whose working memory has to fit max_bytes: the free plan
// (plan_step of the same row tiles) where that fits, else one with as few splits
// and as wide LM-head tiles as it takes, which adds the same products in another
// order. The result may still be too large.
inline StepPlans fit_plan(const ModelShape* m, int M, size_t scratch, const StepPlans& free_plan,
                          size_t max_bytes) {
  const WsLayout w = ws_layout(m, free_plan, M, scratch);
  if (w.total <= max_bytes) return free_plan;
  // what the shared region may take (the FP8 one holds the SwiGLU rows as well)
  const size_t f = m->fp8 ? (size_t)free_plan.rt.rows() * round256(m->cfg.ffn) * 2 : 0;
  const size_t rest = w.total - std::max(w.shared_bytes, (f + 255) / 256 * 256);
  if (rest >= max_bytes) return free_plan;
  return plan_step(m, free_plan.rt, (max_bytes - rest) / 256 * 256, 8);
}

"""The plans of a verify forward and the sizes of its working memory
(csrc/plan.h), checked on the CPU.

* The plan of lopa_verify_forward is the one the planner estimates fastest; the
  fixed working memory of lopa_verify_forward_noalloc has no part in it.
* lopa_verify_forward_noalloc takes that same plan (the same bits) at every shape
  of FITS, and accepts every shape of TIGHT.
* The regions of the working memory that are alive together do not overlap."""
import os
import shutil
import subprocess

import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include "attn_span.h"
#include "plan.h"

// argv: layers hidden heads kv_heads head_dim ffn vocab precision n_branches L
int main(int, char** v) {
  lopa_model_cfg c{};
  int* f[] = {&c.layers, &c.hidden, &c.heads, &c.kv_heads, &c.head_dim, &c.ffn, &c.vocab};
  for (int i = 0; i < 7; ++i) *f[i] = atoi(v[1 + i]);
  ModelShape m;
  m.num_cu = 256;
  m.set(c, atoi(v[8]));
  const int nb = atoi(v[9]), L = atoi(v[10]), M = nb * L;
  const std::vector<StepPlans> plans = all_plans(&m, 2048);
  const StepPlans p = plans[row_tiles(M).index()];
  const size_t scratch = attention_scratch_bytes(nb, L, c.heads, c.kv_heads, c.head_dim);
  const StepPlans q = fit_plan(&m, M, scratch, p, LOPA_NOALLOC_MAX_BYTES);
  const WsLayout w = ws_layout(&m, q, M, scratch);
  auto same = [](const GemmPlan& a, const GemmPlan& b) {
    return a.nb == b.nb && a.tiles == b.tiles && a.splits == b.splits;
  };
  const bool free_plan = same(p.qkv, q.qkv) && same(p.o, q.o) && same(p.gu, q.gu) &&
                         same(p.down, q.down) && same(p.lm, q.lm);
  // regions alive together: the residual stream and abuf with everything; the
  // queries with the partial sums and abuf; the SwiGLU rows with the down
  // projection's partial sums (bf16: read while these are written); the E4M3
  // operands and scales with everything
  const size_t rows = p.rt.rows(), H = c.hidden, q_end = w.qbuf + (size_t)M * c.heads * c.head_dim * 2;
  struct R { size_t a, b; };
  const R x{w.x, w.x + rows * H * 4}, ab{w.abuf, w.abuf + rows * H * 2}, qb{w.qbuf, q_end},
      fb{w.fbuf, w.fbuf + rows * round256(c.ffn) * 2}, sh{w.shared, w.shared + w.shared_bytes};
  const R f8[] = {{w.a8_gu, w.a8_gu + rows * round512(c.hidden)}, {w.a8_dn, w.a8_dn + rows * round512(c.ffn)},
                  {w.sa_gu, w.sa_gu + rows * 4}, {w.sa_dn, w.sa_dn + rows * 4},
                  {w.rowmax_dn, w.rowmax_dn + rows * 4}};
  auto apart = [](R s, R t) { return s.b <= t.a || t.b <= s.a; };
  bool ok = apart(x, ab) && apart(x, qb) && apart(x, fb) && apart(x, sh) && apart(ab, qb) &&
            apart(ab, fb) && apart(ab, sh) && apart(qb, sh) && 3 * w.stats_bytes <= w.shared_bytes &&
            scratch <= w.shared_bytes && partial_bytes(&m, q) <= w.shared_bytes &&
            4 * lm_stats(q) <= w.stats_bytes;
  // the bf16 SwiGLU operand: apart from the partial sums, and its padding columns,
  // zeroed once a forward, past the queries
  if (!m.fp8) ok = ok && apart(fb, sh) && (apart(qb, fb) || q_end <= w.fbuf + rows * (c.ffn / 32 * 32) * 2);
  if (m.fp8)
    for (int i = 0; i < 5; ++i) {
      ok = ok && f8[i].b <= w.total && apart(f8[i], x) && apart(f8[i], ab) && apart(f8[i], qb) &&
           apart(f8[i], fb) && apart(f8[i], sh);
      for (int j = 0; j < i; ++j) ok = ok && apart(f8[i], f8[j]);
    }
  for (const R& r : {x, ab, qb, fb, sh}) ok = ok && r.b <= w.total;
  printf("%d %d %d %d %d %d %d %d %zu\n", free_plan, w.total <= LOPA_NOALLOC_MAX_BYTES, ok, p.qkv.splits,
         p.o.splits, p.down.nb, p.down.splits, p.lm.nb, w.total);
  return 0;
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("amdclang++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(HARNESS)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2512_16229_amd", "csrc"),
                    str(d / "plan.cpp"), "-o", str(d / "plan")], check=True)

    def run(layout, vocab, prec, nb, L, **over):
        c = synth.config(layout, vocab=vocab, **over)
        args = [c[k] for k in ("layers", "hidden", "heads", "kv_heads", "head_dim", "ffn", "vocab")]
        args += [{"bf16": 0, "fp8_mlp": 1, "fp8": 2}[prec], nb, L]
        out = subprocess.run([str(d / "plan"), *map(str, args)], capture_output=True, text=True, check=True)
        keys = ("free", "fits", "apart", "qkv_s", "o_s", "down_nb", "down_s", "lm_nb", "bytes")
        return dict(zip(keys, map(int, out.stdout.split())))
    return run


# (layout, vocabulary, precision, branches, block, QKV splits, down splits): forwards
# of 512 to 768 rows whose working memory lies near the fixed 64 MiB. Fewer splits of
# the down projection (3 instead of 4, 1 instead of 3) leave a third to a half of the
# CUs without a workgroup.
FREE = [("dream7b", 152064, "bf16", 16, 32, 3, 4), ("dream7b", 152064, "bf16", 8, 64, 3, 4),
        ("dream7b", 16384, "bf16", 20, 32, 2, 3), ("dream7b", 16384, "bf16", 10, 64, 2, 3),
        ("dream7b", 16384, "fp8_mlp", 16, 32, 3, 4), ("llada8b", 126464, "bf16", 16, 32, 1, 4),
        ("llada8b", 16384, "fp8", 8, 64, 1, 4)]


@pytest.mark.parametrize("layout,vocab,prec,nb,L,qkv_s,down_s", FREE)
def test_the_fixed_array_does_not_limit_the_plan(harness, layout, vocab, prec, nb, L, qkv_s, down_s):
    r = harness(layout, vocab, prec, nb, L)
    assert (r["qkv_s"], r["down_nb"], r["down_s"]) == (qkv_s, 8, down_s)


# shapes at which lopa_verify_forward_noalloc has the bits of lopa_verify_forward
FITS = [("dream7b", 152064, p, nb, L) for p in ("bf16", "fp8_mlp", "fp8")
        for nb, L in ((1, 32), (8, 32), (16, 16), (4, 64), (1, 256), (16, 32), (8, 64))]
FITS += [("llada8b", 126464, p, nb, L) for p in ("bf16", "fp8_mlp", "fp8")
         for nb, L in ((8, 32), (8, 48), (4, 128))]
FITS += [("llada8b", 16384, "fp8_mlp", 16, 32), ("wide1536", 2048, "bf16", 28, 64),
         ("wide1536", 152064, "bf16", 24, 64), ("wide6144", 2048, "bf16", 15, 33),
         ("tiny", 1024, "bf16", 8, 256), ("small", 3000, "fp8", 8, 256)]


@pytest.mark.parametrize("layout,vocab,prec,nb,L", FITS)
def test_noalloc_takes_the_same_plan(harness, layout, vocab, prec, nb, L):
    r = harness(layout, vocab, prec, nb, L)
    assert r["fits"] and r["free"] and r["apart"], r


# shapes it runs with fewer splits
TIGHT = [("dream7b", 16384, "bf16", 10, 64), ("dream7b", 16384, "bf16", 12, 64),
         ("llada8b", 126464, "bf16", 9, 64), ("wide6144", 2048, "fp8_mlp", 9, 64)]


@pytest.mark.parametrize("layout,vocab,prec,nb,L", TIGHT)
def test_noalloc_accepts_with_fewer_splits(harness, layout, vocab, prec, nb, L):
    r = harness(layout, vocab, prec, nb, L)
    assert r["fits"] and not r["free"] and r["apart"], r


def test_noalloc_refuses_what_cannot_fit(harness):
    assert not harness("tiny", 1024, "bf16", 16, 32, layers=1, ffn=65536)["fits"]
    assert not harness("dream7b", 152064, "bf16", 16, 64)["fits"]

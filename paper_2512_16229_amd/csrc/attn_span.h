// Which keys the attention of a branch covers and how the single-load form cuts
// them into tiles: index arithmetic of attention.hip that a host program can
// compile too, to check every index it yields.
#pragma once

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define ATTN_HD __host__ __device__ __forceinline__
#else
#define ATTN_HD inline
#endif

constexpr int KT = 32;       // keys per tile
constexpr int SL_WAVES = 8;  // wavefronts of a single-load workgroup

// What the rows of branch br see: P cache positions, then Lk keys of their own
// staging; Lr rows. Chained (chain_rows > 0, AttnArgs): branch br is block br of a
// run of blocks whose K / V are in the cache already, and sees the cache up to
// its own end; the last block may be short.
struct AttnSpan {
  int P, Lk, Lr;
};
ATTN_HD AttnSpan attn_span(int P, int L, int chain_rows, int br) {
  if (!chain_rows) return {P, L, L};
  const int r0 = br * L, left = chain_rows - r0, Lr = left < L ? left : L;
  return {P + r0 + Lr, 0, Lr};
}
// tiles of the prefix, and of the prefix and the staging (at least one)
ATTN_HD int prefix_tiles(const AttnSpan& s) { return (s.P + KT - 1) / KT; }
ATTN_HD int key_tiles(const AttnSpan& s) { return prefix_tiles(s) + (s.Lk + KT - 1) / KT; }

// Single-load form: wavefront wv takes tiles t_lo .. t_lo + nt - 1 of T. A kernel
// instance holds the scores of NT tiles, as many as any wavefront of the launch
// has; sl_buffers(NT) K (then V) tiles are in flight.
struct SlRange {
  int t_lo, nt;
};
ATTN_HD SlRange sl_range(int T, int wv) {
  const int lo = wv * T / SL_WAVES;
  return {lo, (wv + 1) * T / SL_WAVES - lo};
}
ATTN_HD constexpr int sl_buffers(int NT) { return NT <= 3 ? NT : 2; }
// Tile of load i. With more tiles than buffers the loads sit under no branch: past
// the wavefront's last tile they take that tile again, and a wavefront without a
// tile takes t_lo, which lies in the range too (t_lo <= 7 T / 8 < T). An early
// block of a chained run has such wavefronts: NT follows the run's last block,
// which may see 25 tiles and more while the first sees one.
ATTN_HD int sl_tile(const SlRange& r, int i) {
  return r.t_lo + (i < r.nt ? i : r.nt > 0 ? r.nt - 1 : 0);
}

// Which keys the attention of a branch covers and how the single-load form cuts
// them into tiles: index arithmetic of attention.hip that a host program can
// compile too, to check every index it yields.
#pragma once
#include <stddef.h>

#include <algorithm>

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
// (selects, no branch: it stands before a kernel's first load)
ATTN_HD AttnSpan attn_span(int P, int L, int chain_rows, int br) {
  const int r0 = br * L, left = chain_rows - r0, Lr = chain_rows && left < L ? left : L;
  return {P + (chain_rows ? r0 + Lr : 0), chain_rows ? 0 : L, Lr};
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

// Grouped form: key splits before the per-call caps, enough workgroups for the
// chip's 256 CUs, at most 16
inline int group_splits(int nb, int Hkv) {
  return std::min(16, std::max(1, (256 + Hkv * nb - 1) / (Hkv * nb)));
}
// bytes of AttnArgs::scratch that let the grouped form run with its full key
// splits for nb branches of L rows at any prefix (0: the shape never takes it)
inline size_t attention_scratch_bytes(int nb, int L, int Hq, int Hkv, int d) {
  const int G = Hkv > 0 ? Hq / Hkv : 0;
  if (L > 32 || G < 2 || G > 8) return 0;
  const size_t rows = (size_t)nb * Hq * L;
  return rows * group_splits(nb, Hkv) * (2 + (size_t)d) * 4;
}

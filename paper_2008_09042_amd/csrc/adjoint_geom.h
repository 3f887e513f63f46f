// How the dense adjoint's work is split (stream_adjoint.h; host code without HIP).
#pragma once

#include <cstddef>
#include <cstdint>

namespace mx {

constexpr int ADJ_WAVES = 8;  // per workgroup

struct AdjGeom {
  int JB, AKB, jgs;  // 16-coil blocks and 16-column blocks per wave, coil groups
  int kwl, ks;       // log2 of the column groups per workgroup (0 to 2), workgroups per row chunk along K
  int64_t chunk;     // rows per workgroup
  int nchunk;
};

// Waves: two column groups where K has two, and row groups.  A workgroup over all of K (up to
// eight groups) left its partials, one per row chunk, to be most of the traffic of a short
// basis, and each wave a step or two: 64 x 64, 17 coils, 300 columns, BF16-split 20.7 -> 12.1 us,
// FP32 23.1 -> 14.5; 128 x 128, 32 coils, 512 columns 35.4 -> 23.4; 256 x 256, 32 coils, 200
// columns 32.8 -> 28.4.  One group per workgroup reads h once per 64 columns: better up to
// 256 x 256 (26.9), worse beyond (512 x 512, 16 coils, 100 columns 44.3 -> 52.3).
// Three or four groups of many rows take one workgroup over all of K: two of them would be
// uneven, a whole workgroup for a few last columns, and read h twice (two groups -> four,
// 512 x 512, 3 coils, 130 columns 67.5 -> 52.9 us; 1000 x 800, 16 coils, 130 columns 233 -> 185;
// but 256 x 256, 32 coils, 200 columns 30.2 -> 34.6).
// Row chunks: a workgroup per compute unit over all coil and column groups (two where the
// tiles are small enough that two share one), or as few rounds of that as leave at most a tenth
// of the last one idle, at least one step of every row group, and no more than max_chunks (0: no
// limit).  Never fewer than 32 chunks, as it was, gave 10 column groups 320 workgroups: 192 x 192,
// 33 coils, 600 columns, FP32 167 -> 118 us, 400 x 400, 100 coils, 258 columns 674 -> 439.
inline AdjGeom adj_geom(int64_t N, int64_t K, int J, int max_chunks) {
  AdjGeom a;
  const int nkb = (int)((K + 15) / 16), njb = (J + 15) / 16;
  a.JB = njb == 1 ? 1 : njb == 2 ? 2 : 4;
  a.jgs = (njb + a.JB - 1) / a.JB;
  a.AKB = a.JB < 4 && nkb > 2 ? 4 : 2;
  const int groups = (nkb + a.AKB - 1) / a.AKB;
  a.kwl = (groups == 3 || groups == 4) && N >= 131072 ? 2 : groups > 1 ? 1 : 0;
  a.ks = (groups + (1 << a.kwl) - 1) >> a.kwl;
  const int64_t step = (int64_t)16 * (ADJ_WAVES >> a.kwl);
  const int64_t slots = a.JB == 1 ? 512 : 256, per = (int64_t)a.jgs * a.ks;
  int64_t rounds = 1;
  while (10 * (slots * rounds / per) * per < 9 * slots * rounds) ++rounds;
  int64_t want = slots * rounds / per;
  if (max_chunks > 0 && want > max_chunks) want = max_chunks;
  a.chunk = (N + want - 1) / want;
  a.chunk = (a.chunk + step - 1) / step * step;
  a.nchunk = (int)((N + a.chunk - 1) / a.chunk);
  return a;
}

}  // namespace mx

// Chunks of the TOA pass and the waves that share one: host arithmetic without
// the HIP runtime.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace pt {

constexpr int kTile = 16;          // TOAs per MFMA row tile
constexpr int kToaMaxWaves = 8;    // waves that share a chunk, at most
// Zeros past the last TOA of the per-TOA arrays.  A wave loads the tile after its
// own (16 times the waves of its chunk further on) before it looks whether there
// is one: from a tile that starts at the last TOA, up to 16 kToaMaxWaves + 15 on.
constexpr int kToaPad = kTile * kToaMaxWaves + kTile - 1;

struct ToaChunks {
  std::vector<int32_t> psr, begin, end;   // of each chunk
  std::vector<int32_t> first;             // [n_psr + 1] first chunk of a pulsar
  int max_tiles = 0;                      // of the longest chunk
};

// Every pulsar in chunks of about `tpc` tiles (tile-aligned, at least one).
inline ToaChunks cut_chunks(const int64_t *off, int n_psr, int tpc) {
  ToaChunks c;
  for (int p = 0; p < n_psr; ++p) {
    const int64_t b = off[p], e = off[p + 1], tiles = (e - b + kTile - 1) / kTile;
    const int64_t nch = std::max<int64_t>(1, (tiles + tpc - 1) / tpc);
    c.first.push_back((int32_t)c.psr.size());
    for (int64_t i = 0; i < nch; ++i) {
      const int64_t t0 = (i * tiles) / nch, t1 = ((i + 1) * tiles) / nch;
      c.psr.push_back(p);
      c.begin.push_back((int32_t)(b + kTile * t0));
      c.end.push_back((int32_t)std::min<int64_t>(e, b + kTile * t1));
      c.max_tiles = std::max(c.max_tiles, (int)(t1 - t0));
    }
  }
  c.first.push_back((int32_t)c.psr.size());
  return c;
}

// Waves per workgroup of the TOA pass: those that ptafs_set_tuning gave (tuned), or
// without it one, and more for a data set of few and long chunks.  The chunk's
// waves are combined in LDS, so neither the chunks nor the partials change.  The
// rule does not look at the number of chains, on which a chain's result does not
// depend: its lines lie where up to 256 chains are not slower for it, by 256
// compute units.  Microseconds a launch at 16, 128 and 256 chains with 1, 2, 4 and
// 8 waves a chunk, 30 harmonics with DM:
//   chunks of 16 tiles:   6   41 26 20 17   42 26 20 18   42 27 21 18
//                        31   41 26 20 17   43 28 22 19   46 43 30 33
//                        63   41 27 20 18   45 44 30 32   78 47 61 58
//                        80   42 27 21 18   46 45 39 45   78 67 63 72
//                       127   42 27 21 18   77 47 60 58   82 92 96 107
//              8 tiles:  31   24 17 15 13   26 19 17 15   27 27 24 26
//                        80   25 18 16 14   27 28 27 33   45 47 45 51
//              4 tiles:  16   15 13 13      16 13 14      16 14 14
//                        63   15 13 14      18 19 17      27 22 30
// Beyond 256 chains more waves still gain with 16 chunks (1024 chains: 78 with one,
// 59 with eight) and cost with 31 (82, 110).
inline int toa_waves(bool tuned, int waves, int max_chunk_tiles, int n_chunks, int n_cu) {
  if (tuned) return waves;
  if (max_chunk_tiles >= 8) return 8 * n_chunks < n_cu ? 8 : 3 * n_chunks < n_cu ? 4 : 1;
  return max_chunk_tiles >= 4 && 16 * n_chunks <= n_cu ? 2 : 1;
}

}  // namespace pt

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

// Waves per workgroup of the TOA pass: the tuning's, and up to eight for a data
// set whose chunks would otherwise have fewer waves than there are compute
// units by half (in one block of 16 chains: the rule must not look at the number
// of chains, on which a chain's result does not depend), as long as every wave of
// the longest chunk has a tile.  The chunk's waves are combined in LDS, so
// neither the chunks nor the partials change.  Three pulsars of 500 TOAs (6
// chunks of 16 tiles): 14.4 us a launch with one wave a chunk, 6.9 with eight;
// with a continuous wave (33 chains) 20 and 12.8.  Beyond that line more waves
// cost where there are many chains: 22 pulsars of 750 TOAs, 193 chains and chunks
// cut to fill the device (about 150), 123 us an evaluation with one wave a chunk,
// 126 with two; 192 chunks of 67 pulsars at 64 chains take 13 us more with eight
// waves than with the four they are tuned to.
inline int toa_waves(int tuned, int max_chunk_tiles, int n_chunks, int n_cu) {
  int w = tuned;
  while (w < kToaMaxWaves && 2 * w <= max_chunk_tiles && 2 * w * n_chunks < n_cu) w *= 2;
  return w;
}

}  // namespace pt

// Arithmetic of a selection's workspace, without device code: the kernels, the host and a CPU test share it.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace lava {

constexpr size_t kAlign = 256;
constexpr size_t align_up(size_t x, size_t a = kAlign) { return (x + a - 1) / a * a; }

constexpr int kSelThreads = 1024;   // few, large workgroups: a wait for the others and a histogram merge cost per workgroup
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelBins = 2048;      // a selection region's histogram area is 3 * kSelBins words
constexpr int kSelStateWords = 8;   // words of its state block (cleared together with its histograms)
constexpr int kSegWords = 64;       // keys of the threshold's interval a workgroup may contribute, per key a lane holds
constexpr int kMostKeys = 12;       // keys per lane of the one-launch selection: 2, 4, 8 or this

struct SelectWorkspace {
  size_t off_hist;        // uint32 [3 * kSelBins]: the histograms, then the exchange words of the one-launch selection
  size_t off_state;       // SelectState
  size_t off_blk;         // uint32 [blk_words]: a segment of keys per workgroup of the one-launch selection, or the
                          // step launches' [2][workgroups] counts of keys above / equal to the threshold
  int n_blocks;
  size_t blk_words;
  size_t bytes;
};

// Layout of a selection's workspace for `total` entries (also evaluated at compile time, for the built-in
// scratch array of lava_select_topk_static).
constexpr SelectWorkspace select_layout(int64_t total) {
  constexpr int64_t kChunk = kSelThreads * 16;
  SelectWorkspace w{};
  w.n_blocks = (int)((total + kChunk - 1) / kChunk);
  if (w.n_blocks < 1) w.n_blocks = 1;
  size_t off = 0;
  w.off_hist = off;  off += align_up(sizeof(uint32_t) * 3 * kSelBins);
  w.off_state = off; off += align_up(sizeof(uint32_t) * kSelStateWords);
  // two counts per workgroup for the step launches; the one-launch selection's segments: kSegWords for every 1024 entries
  constexpr int kRegionBlocks = 1024;
  w.blk_words = 2 * (size_t)w.n_blocks;
  const size_t fused = (size_t)(w.n_blocks < kRegionBlocks ? w.n_blocks : kRegionBlocks) * (16 * kSegWords + 1);
  if (fused > w.blk_words) w.blk_words = fused;
  w.off_blk = off;   off += align_up(sizeof(uint32_t) * w.blk_words);
  w.bytes = off;
  return w;
}

// Workgroups of the one-launch selection with `keys` keys per lane.
constexpr int64_t workgroups_for(int64_t total, int keys) {
  const int64_t chunk = (int64_t)kSelThreads * keys, nb = (total + chunk - 1) / chunk;
  return nb < 1 ? 1 : nb;
}

// Words of one workgroup's segment, where `workgroups` of them share a region of blk_words: kSegWords per key, or an
// equal share where that is less.  (The region is laid out by 16384 entries, which 2, 4 and 8 keys per lane divide and 12
// do not: a last, partly filled workgroup more than the region has whole segments for: 1048576 entries, 86 x 768 words
// of 65600, get 762 each.)
constexpr unsigned int segment_words(int keys, int64_t workgroups, size_t blk_words) {
  const size_t most = (size_t)kSegWords * keys, share = blk_words / (size_t)workgroups;
  return (unsigned int)(share < most ? share : most);
}

// Entries of a wavefront are base .. base + span - 1, and totals go up to 2^31 - 1: base + span may be 2^31, so it
// is never formed.
constexpr bool span_complete(int base, int span, int total) { return base <= total - span; }   // every entry exists
constexpr bool in_span(int p, int base, int span) { return p >= base && p - base < span; }      // p, base >= 0

}  // namespace lava

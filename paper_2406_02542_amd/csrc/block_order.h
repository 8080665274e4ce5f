// Which work a block of the one-block-per-head launches does: plain arithmetic, also compiled for the host.
#pragma once

#ifdef __HIPCC__
#define LOKI_HOST_DEVICE __host__ __device__
#else
#define LOKI_HOST_DEVICE
#endif

namespace loki {

// Ragged batches: the rank by length, longest first, of the sequence at place `pos` of the launch.
// The first half of the places takes the longest sequences in descending order, the second half the
// rest in ascending order; no sequence (-1) belongs to a place past the last one.
LOKI_HOST_DEVICE constexpr int paired_rank(int pos, int n_seq) {
  const int half = (n_seq + 1) / 2;
  return pos < half ? pos : pos < n_seq ? n_seq - 1 - (pos - half) : -1;
}

// Launches of G heads per unit, padded to a multiple of 8 units: a unit's heads are blocks 8 apart.
// The place of block's unit among the units, or -1 for the padding; its head is grouped_head.
LOKI_HOST_DEVICE constexpr int grouped_slot(int block, int G, int units) {
  const int slot = block / 8 / G * 8 + block % 8;
  return slot < units ? slot : -1;
}
LOKI_HOST_DEVICE constexpr int grouped_head(int block, int G) { return block / 8 % G; }

}  // namespace loki

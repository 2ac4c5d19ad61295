// Host-side launchers of the channel-mutation kernels (channel_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.hpp"

namespace mca {

// Hidden widths the channel kernels take (every hidden layer the same).
inline bool channel_width_ok(int w) { return w == 256 || w == 512 || w == 1024; }
// Segments of the samples, listed apart, and tile sums per channel.
int channel_segments(int64_t n_samples);
int channel_tiles(int64_t n_samples, int w, int n_layers);

// The samples whose change goes past the path's units, per channel of
// list_group(), or of the largest batch (N entries each): the sample, the changed
// activation and the path unit's new one, and the layer the change enters; the
// lists' lengths (two per channel and segment of the samples) and the first tile of
// each (one more).
struct ChannelLists {
  int* rows;
  float* d;
  float* ap;
  int* f;
  int* cnt;
  int* first;
};

// Draws channels k = 0..K-1 of step t (use_dev_t: st->t) into ch, with
// their acceptance data in aux and a placeholder record per candidate in
// cands (the shared selection reads one).
hipError_t launch_channel_propose(const NetDev& net, uint64_t t, bool use_dev_t,
                                  const DevState* st, int K, mca_channel* ch, mca_cand* cands,
                                  Aux* aux, hipStream_t s, mca_channel* host = nullptr);
// The same acceptance data for K channels given by the caller (threshold 0).
hipError_t launch_channel_prepare(const NetDev& net, mca_channel* ch, int K,
                                  mca_cand* cands, Aux* aux, hipStream_t s,
                                  const mca_channel* host = nullptr);
// k_mode -2: partial[k * nchan + tile] for every channel k < K; -1: commit
// st->chosen (nothing when -1); >= 0: commit that channel.  A commit moves
// every cached field and writes the path's weights, the loss and the count.
hipError_t launch_channel(const NetDev& net, const mca_channel* ch, const Aux* aux, int K,
                          const ChannelLists& lists, float* partial, int nchan, int k_mode,
                          DevState* st, const double* dL, hipStream_t s);

}  // namespace mca

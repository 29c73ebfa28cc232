// Launchers of the stride-1 convolution kernels that form fp32 products from
// bf16 parts (conv_split.hip).
#pragma once

#include "common.h"

namespace oc {

// Shape of k_conv_sp3 for a K = 3 layer of G sibling groups, kk reduction and
// nn output channels (multiples of 4, kk >= 16): WN blocks of 16 output
// channels and GPB sibling groups per workgroup tile.
struct Sp3Cfg {
  int wn, gpb, splits;
};
Sp3Cfg sp3_pick(int64_t G, int kk, int nn);

// Where the pooled forward writes: pooled rows of depth l-1 and switches.
struct Sp3Pool {
  float* y;
  uint8_t* sw;
};

// out [N_l][nn] = the stride-1, K = 3 convolution of x [N_l][kk] (flip: the
// input gradient, weights w [27][nn][kk]); with cfg.splits > 1 the partial
// sums of the reduction's 16-channel chunks go to part[split][N_l][nn]
// instead.  pool (cfg.splits == 1, not flip): the 2x2x2 max-pool of the
// result is written and out is not.
void sp3_launch(const oc_octree* t, int l, const Sp3Cfg& cfg, bool flip, const float* x, int kk,
                const float* w, int nn, float* out, int relu, float* part, const Sp3Pool* pool,
                hipStream_t s);

// Kernel name with template arguments.
void sp3_name(const oc_octree* t, int l, const Sp3Cfg& cfg, bool flip, bool pooled, int kk, char* buf,
              size_t n);

// Partial sums part[nchunks][27][cin][cout] of the K = 3 weight gradient over
// chunks of gchunk sibling groups (cin >= 16, cin and cout multiples of 4),
// nbn = 1 or 2 blocks of 16 columns per workgroup of 16 channels.
void dws_launch(const oc_octree* t, int l, int nbn, int64_t gchunk, int64_t nchunks, const float* x,
                int cin, const float* dy, int cout, float* part, hipStream_t s);
void dws_name(const oc_octree* t, int l, int nbn, int cin, int cout, char* buf, size_t n);

}  // namespace oc

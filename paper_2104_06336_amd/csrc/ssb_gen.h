// The column transform fused with Eq. 3 at any scan length (ssb_gen.hip): layout and launcher.
#pragma once

#include "fft_generic.h"
#include "ssb_fused.h"

namespace stem {

// threads of a workgroup: the last pass has at most one butterfly per thread
inline int gsum_threads(int ny) { return ny > 2048 ? 512 : 256; }

// Pixel groups: about 2048 workgroups for a sum over all pixels at once (the GPU holds 768: enough
// rounds to even out columns of few pairs), half of that when the pixels come in chunks, whose
// launches are short and each reread the partial sums; at most one pixel per group, 64 MB of partials.
inline int gsum_groups(int ny, int nx, int pixels, bool chunked) {
  const int nc = nx / 2 + 1;
  int64_t g = ((chunked ? 1024 : 2048) + nc / 2) / nc;
  const int64_t gmax = (64ll << 20) / ((int64_t)ny * nx * 8);
  g = g > gmax ? gmax : g;
  g = g > pixels ? pixels : g;
  return (int)(g < 1 ? 1 : g);
}

// waves of a launch (each writes its pair counter)
inline int64_t gsum_waves(int ny, int nx, int ngroups) {
  return (int64_t)(nx / 2 + 1) * ngroups * (gsum_threads(ny) / 64);
}

// Pixels a workgroup transforms together and the plan of ny: at least one at every length the library
// transforms, 0 if ny has no plan.
int gsum_rows(int ny, GPlan& p);

// The sum over the pixels [a.k0, a.k1), whose row-transformed columns are at a.X, in a.ngroups groups;
// pwrite: also store the double-overlap values as the pruned array.
int launch_gsum(int ny, const YArgs& a, const Optics& o, int chi0, bool pwrite, hipStream_t s);

}  // namespace stem

// Detector / scan geometry shared by host and device code: exact integer division by an
// invariant divisor, the kept-bin predicate and the per-row description of the kept set.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "stem4d.h"

namespace stem {

// floor(n / d) for 0 <= n < 2^31 and 1 <= d < 2^31 by one 64-bit multiply and shift:
// with l = ceil(log2 d), m = ceil(2^(31+l) / d) the quotient is (n*m) >> (31+l)
// (Granlund & Montgomery, "Division by invariant integers using multiplication", Thm 4.2).
struct Magic {
  uint64_t m;
  uint32_t shift;
  uint32_t d;
};

inline Magic make_magic(uint32_t d) {
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  const unsigned __int128 num = (unsigned __int128)1 << (31 + l);
  uint64_t m = (uint64_t)((num + d - 1) / d);
  return Magic{m, 31 + l, d};
}

__host__ __device__ __forceinline__ uint32_t magic_div(uint32_t n, const Magic& mg) {
  return (uint32_t)(((uint64_t)n * mg.m) >> mg.shift);
}

// Row of a detector pixel, k div W.  Detectors of up to 2^24 pixels take one full-rate 24-bit
// multiply (D24): ((k << sh) m) >> 32 with m = ceil(2^(32-sh) / W) < 2^24, exact while k (m W - 2^(32-sh)) <
// 2^(32-sh) for every pixel.  Others multiply in 64 bits.  mbin: division of a coordinate by the binning,
// ((x << 8) mbin) >> 32 with mbin = ceil(2^24 / bin) (D24, exact while x bin < 2^24), else (x mbin) >> 32 with
// ceil(2^32 / bin); 0 for bin = 1.
struct PixDiv {
  Magic mg;
  uint32_t m, sh, mbin, d24;
};

inline PixDiv make_pixdiv(int32_t W, int32_t H, int32_t bin) {
  PixDiv p{make_magic((uint32_t)W), 0u, 0u, 0u, 0u};
  const uint64_t npix = (uint64_t)W * (uint64_t)H;
  for (uint32_t sh = 0; sh <= 8 && (npix << sh) <= (1ull << 24) && W < 32768 && H < 32768; ++sh) {
    const uint64_t one = 1ull << (32 - sh), m = (one + W - 1) / W;
    if (m >= (1ull << 24) || (npix - 1) * (m * W - one) >= one) continue;
    if ((uint64_t)(W > H ? W : H) * (uint64_t)bin >= (1ull << 24)) break;
    p.m = (uint32_t)m;
    p.sh = sh;
    p.d24 = 1u;
    break;
  }
  if (bin > 1) p.mbin = p.d24 ? (uint32_t)(((1ull << 24) + bin - 1) / bin) : (uint32_t)(((1ull << 32) + bin - 1) / bin);
  return p;
}

template <bool D24>
__device__ __forceinline__ uint32_t pix_row(uint32_t k, const PixDiv& p) {
  if constexpr (D24) return (uint32_t)(((uint64_t)((k << p.sh) & 0xffffffu) * (p.m & 0xffffffu)) >> 32);
  else return magic_div(k, p.mg);
}
// k - row W
template <bool D24>
__device__ __forceinline__ uint32_t pix_col(uint32_t k, uint32_t row, const PixDiv& p) {
  if constexpr (D24) return k - (uint32_t)__umul24(row, p.mg.d);
  else return k - row * p.mg.d;
}
// x div bin
template <bool D24>
__device__ __forceinline__ uint32_t pix_bin(uint32_t x, const PixDiv& p) {
  if (!p.mbin) return x;
  if constexpr (D24) return (uint32_t)(((uint64_t)((x << 8) & 0xffffffu) * (p.mbin & 0xffffffu)) >> 32);
  else return __umulhi(x, p.mbin);
}

// The whole 16-byte lines of an int32 array at address base that hold at least one of its entries [e0, e1):
// n of them, the first starting at entry `first` (up to three before e0).  None for an empty range.
struct Lines {
  int64_t first, n;
};
__host__ __device__ __forceinline__ Lines lines_of(uintptr_t base, int64_t e0, int64_t e1) {
  const int64_t first = e0 - (int64_t)(((base + 4 * (uintptr_t)e0) & 15) >> 2);
  return Lines{first, e1 > e0 ? (e1 - first + 3) >> 2 : 0};
}

// Centre of bin index j along an axis, relative to the zero-frequency pixel c, in unbinned
// pixels: b*j + (b-1)/2 - c.  Exact in double (multiples of 1/2 far below 2^53).
__host__ __device__ __forceinline__ double bin_centre(int b, int j, int c) {
  return (double)(b * j - c) + 0.5 * (double)(b - 1);
}

// Kept-bin predicate: centre strictly inside the bright-field disk, |Kc|^2 < r2.
__host__ __device__ __forceinline__ bool bin_kept(double kx, double ky, double r2) {
  return kx * kx + ky * ky < r2;
}

// The kept bins of one bin row form a contiguous run [lo, hi) (a disk meets a line in an
// interval).  Binary searches with the exact predicate.
__host__ __device__ inline void kept_run(int b, int by, int nbx, int cx, int cy, double r2, int& lo,
                                         int& hi) {
  const double ky = bin_centre(b, by, cy);
  // the bin closest to the axis x = 0 (the minimiser of |Kc_x|)
  int best = 0;
  {
    int a = 0, z = nbx - 1;  // last index with centre < 0, if any
    if (bin_centre(b, 0, cx) >= 0.0) {
      best = 0;
    } else {
      while (a < z) {
        int mid = (a + z + 1) / 2;
        if (bin_centre(b, mid, cx) < 0.0) a = mid; else z = mid - 1;
      }
      best = a;
      if (a + 1 < nbx && -bin_centre(b, a, cx) > bin_centre(b, a + 1, cx)) best = a + 1;
    }
  }
  if (!bin_kept(bin_centre(b, best, cx), ky, r2)) {
    lo = hi = 0;
    return;
  }
  int a = 0, z = best;  // first kept in [0, best]
  while (a < z) {
    int mid = (a + z) / 2;
    if (bin_kept(bin_centre(b, mid, cx), ky, r2)) z = mid; else a = mid + 1;
  }
  lo = a;
  a = best;
  z = nbx - 1;  // last kept in [best, nbx)
  while (a < z) {
    int mid = (a + z + 1) / 2;
    if (bin_kept(bin_centre(b, mid, cx), ky, r2)) a = mid; else z = mid - 1;
  }
  hi = a + 1;
}

// Per bin row: first kept pixel number and the run [lo, hi) of kept bx.
struct RowRun {
  int32_t start, lo, hi, pad;
};

}  // namespace stem

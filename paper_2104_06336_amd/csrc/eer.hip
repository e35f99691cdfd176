// Event ingest and per-frame event reductions on linear-index EER (Sec. II, Table 1, Eq. 4).
//
//  k_validate       : range check of event indices and monotonicity of frame offsets.
//  k_com            : per-frame count and exact integer first moments -> centre of mass.
//  k_bin            : per-frame binned, cropped counts into the dense cube D[kd][f].
//
// Frame blocks: a workgroup owns a run of consecutive frames; their events are one contiguous
// CSR slice, read with coalesced 16-byte loads: staged in LDS for the per-frame sums of k_com,
// streamed with an LDS map event -> frame for the counts of k_bin.
#include <cmath>
#include <type_traits>

#include "common.h"
#include "geom.h"
#include "kernels.h"
#include "optics.h"
#include "trace.h"

namespace stem {

constexpr int kComThreads = 256;
constexpr int kComFrames = 256;  // of the run-length re-coding: thread t takes frame t

// ---------------------------------------------------------------------------------------------
// validation

// Only events inside [lo_bound, hi_bound), the range the caller guarantees to be allocated, are looked at; offsets
// outside it are reported, never followed.  They are loaded by whole 16-byte lines, each of which holds at least
// one of them (so it lies in the array's pages; the other entries of a line are masked), four in flight per thread.
__global__ void __launch_bounds__(256) k_validate(const int32_t* __restrict__ idx,
                                                  const int64_t* __restrict__ off, int64_t frame0,
                                                  int64_t n_frames, int64_t n_events, int exact_count,
                                                  int64_t lo_bound, int64_t hi_bound, int32_t npix,
                                                  int32_t* status) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nthr = (int64_t)gridDim.x * blockDim.x;
  const int64_t e0 = off[frame0];
  const int64_t e1 = off[frame0 + n_frames];
  int32_t bits = 0;
  const bool bounds_ok = e0 >= lo_bound && e0 <= e1 && e1 <= hi_bound;
  if (tid == 0 && (!bounds_ok || (exact_count && e1 - e0 != n_events))) bits |= STEM_EOFFSETS;
  for (int64_t f = tid; f < n_frames; f += nthr)
    if (off[frame0 + f + 1] < off[frame0 + f]) bits |= STEM_EOFFSETS;
  if (bounds_ok) {
    const Lines ln = lines_of((uintptr_t)idx, e0, e1);
    const int64_t al = ln.first, ng = ln.n;
    for (int64_t g0 = tid; g0 < ng; g0 += 4 * nthr) {
      int4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t g = g0 + u * nthr;
        v[u] = g < ng ? *(const int4*)(idx + al + 4 * g) : make_int4(0, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t e = al + 4 * (g0 + u * nthr);
        const bool bad[4] = {(uint32_t)v[u].x >= (uint32_t)npix, (uint32_t)v[u].y >= (uint32_t)npix,
                             (uint32_t)v[u].z >= (uint32_t)npix, (uint32_t)v[u].w >= (uint32_t)npix};
        if (bad[0] | bad[1] | bad[2] | bad[3]) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (bad[q] && e + q >= e0 && e + q < e1) bits |= STEM_ERANGE;
        }
      }
    }
  }
  int32_t wbits = bits;
  for (int o = 32; o > 0; o >>= 1) wbits |= __shfl_xor(wbits, o);
  if ((threadIdx.x & 63) == 0 && wbits) report(status, wbits);
}

// ---------------------------------------------------------------------------------------------
// block-local frame lookup shared by the event-parallel kernels

// Loads the block's offsets relative to its first event.  Returns false (and reports) when
// the block holds 2^30 events or more, which the 32-bit relative offsets cannot address.
__device__ __forceinline__ bool load_rel_offsets(const int64_t* __restrict__ off, int64_t fb, int nf,
                                                 int32_t* s_rel, int64_t* s_base, int32_t* status) {
  const int64_t base = off[fb];
  const int64_t span = off[fb + nf] - base;
  if (span >= (1ll << 30)) {
    if (threadIdx.x == 0) report(status, STEM_EOVERFLOW);
    return false;
  }
  for (int i = threadIdx.x; i <= nf; i += blockDim.x) s_rel[i] = (int32_t)(off[fb + i] - base);
  if (threadIdx.x == 0) *s_base = base;
  return true;
}

// ---------------------------------------------------------------------------------------------
// Staging of a workgroup's events in LDS: the events [a0, a0 + n) (absolute indices, n <= WIN)
// are copied as whole 16-byte lines from the aligned position at or below a0; s[sh + j] then holds
// event a0 + j (sh < 4 is returned).  Every line holds at least one of the events, so it lies in
// the event array's pages; its other entries land outside [sh, sh + n) and are never read.  Each
// thread issues kStageGroups loads before its LDS stores: a window takes one round.
constexpr int kComWin = 12288;  // the run-length re-coding's window
constexpr int kSumWin = 6144;   // and that of the per-frame sums

template <int WIN>
__device__ __forceinline__ int stage_events(const int32_t* __restrict__ idx, int64_t a0, int n, int32_t* s) {
  constexpr int kStageGroups = WIN / (4 * kComThreads);
  const int sh = (int)((((uintptr_t)(idx + a0)) & 15) >> 2);
  const int32_t* ib = idx + (a0 - sh);
  const int ng = (n + sh + 3) >> 2;
  for (int c0 = threadIdx.x; c0 < ng; c0 += kComThreads * kStageGroups) {
    int4 v[kStageGroups];
#pragma unroll
    for (int u = 0; u < kStageGroups; ++u) {
      const int c = c0 + u * kComThreads;
      v[u] = c < ng ? *(const int4*)(ib + 4 * c) : make_int4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < kStageGroups; ++u) {
      const int c = c0 + u * kComThreads;
      if (c < ng) *(int4*)&s[4 * c] = v[u];
    }
  }
  return sh;
}

// ---------------------------------------------------------------------------------------------
// Per-frame sums (centre of mass, annuli): a workgroup owns kComThreads / FT consecutive frames, whose events
// are staged in LDS in windows of kSumWin (coalesced 16-byte loads); the FT threads of a frame take its
// events in turn and add their sums by lane exchange.  With one thread per frame, 256 frames and windows of
// 12288 events a workgroup, a 256 x 256 scan made one workgroup per compute unit and three windows each, and a
// wave ran as long as its longest frame.  Centre of mass, one MI355X: 256 x 256 (100 events a frame) 14
// instead of 29 us, 512 x 512 (60) 15 instead of 25 us, 1024 x 1024 (40) 42 instead of 46 us (4.6 TB/s, about
// the rate of a copy); two annuli at 1024 x 1024 41 instead of 51 us.
//
// FT is 4, and 2 from 2^19 frames on, where there are workgroups enough (1024 x 1024: 50 us with 4).
inline int frame_threads(int64_t n_frames) { return n_frames < (1 << 19) ? 4 : 2; }

// The frames' offsets into s_off; false (reported) when the block holds 2^30 events or more, which the 32-bit
// relative positions cannot address.
__device__ __forceinline__ bool load_offsets(const int64_t* __restrict__ off, int64_t fb, int nf, int64_t* s_off,
                                             int32_t* status) {
  if ((int)threadIdx.x <= nf) s_off[threadIdx.x] = off[fb + threadIdx.x];
  __syncthreads();
  if (s_off[nf] - s_off[0] < (1ll << 30)) return true;
  if (threadIdx.x == 0) report(status, STEM_EOVERFLOW);
  return false;
}

// f(k) for the events of the thread's frame in the window's LDS positions [lo, hi): every FT-th from the
// thread's own, four read ahead
template <int FT, typename F>
__device__ __forceinline__ void frame_events(const int32_t* s_ev, int lo, int hi, int part, F&& f) {
  int e = lo + part;
  for (; e + 3 * FT < hi; e += 4 * FT) {
    int32_t k[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) k[j] = s_ev[e + j * FT];
#pragma unroll
    for (int j = 0; j < 4; ++j) f(k[j]);
  }
  for (; e < hi; e += FT) f(s_ev[e]);
}

template <bool D24, int FT>
__global__ void __launch_bounds__(kComThreads) k_com(const int32_t* __restrict__ idx,
                                                     const int64_t* __restrict__ off,
                                                     int64_t frame0, int64_t n_frames, PixDiv div,
                                                     int32_t cx, int32_t cy, int32_t npix,
                                                     int64_t nplane, double* __restrict__ com64,
                                                     float* __restrict__ com32,
                                                     int32_t* __restrict__ counts,
                                                     int32_t* status) {
  constexpr int kSumFrames = kComThreads / FT;
  __shared__ __align__(16) int32_t s_ev[kSumWin + 8];
  __shared__ int64_t s_off[kSumFrames + 1];
  const int f = threadIdx.x / FT, part = threadIdx.x % FT;
  const int64_t fb = frame0 + (int64_t)blockIdx.x * kSumFrames;
  const int64_t left = frame0 + n_frames - fb;
  const int nf = (int)(left < kSumFrames ? left : kSumFrames);
  if (!load_offsets(off, fb, nf, s_off, status)) return;
  const int64_t base = s_off[0];
  const int span = (int)(s_off[nf] - base);
  const int lo_f = f < nf ? (int)(s_off[f] - base) : 0, hi_f = f < nf ? (int)(s_off[f + 1] - base) : 0;
  int64_t sx = 0, sy = 0;
  int32_t bad = 0;
  for (int w0 = 0; w0 < span; w0 += kSumWin) {
    const int wn = span - w0 < kSumWin ? span - w0 : kSumWin;
    if (w0 > 0) __syncthreads();
    const int sh = stage_events<kSumWin>(idx, base + w0, wn, s_ev);
    __syncthreads();
    const int lo = (lo_f > w0 ? lo_f : w0) - w0 + sh;
    const int hi = (hi_f < w0 + wn ? hi_f : w0 + wn) - w0 + sh;
    // out-of-range indices are counted (and reported) and contribute nothing; no branches.  With the rows
    // ky of the indices k, the columns' sum is the sum of k less W times the sum of ky, here modulo
    // 2^32: a window's columns and rows sum to less (kSumWin W, kSumWin H < 2^32 for sides below 2^18;
    // larger ones sum in 64 bits).
    using S = std::conditional_t<D24, uint32_t, uint64_t>;
    S tk = 0, tr = 0;
    uint32_t nin = 0, n = 0;
    frame_events<FT>(s_ev, lo, hi, part, [&](int32_t k) {
      const bool in = (uint32_t)k < (uint32_t)npix;
      ++n;
      nin += in ? 1u : 0u;
      const uint32_t kk = in ? (uint32_t)k : 0u;
      tk += kk;
      tr += pix_row<D24>(kk, div);
    });
    if (nin != n) bad = STEM_ERANGE;
    const S tc = tk - tr * (S)div.mg.d;
    sx += (int64_t)tc - (int64_t)cx * nin;
    sy += (int64_t)tr - (int64_t)cy * nin;
  }
#pragma unroll
  for (int o = 1; o < FT; o <<= 1) {
    sx += __shfl_xor(sx, o);
    sy += __shfl_xor(sy, o);
  }
  if (f < nf && part == 0) {
    const int64_t fr = fb + f;
    const int64_t n = hi_f - lo_f;
    const double x = n > 0 ? (double)sx / (double)n : 0.0;
    const double y = n > 0 ? (double)sy / (double)n : 0.0;
    if (com64) {
      com64[fr] = x;
      com64[nplane + fr] = y;
    }
    if (com32) {
      com32[fr] = (float)x;
      com32[nplane + fr] = (float)y;
    }
    if (counts) counts[fr] = (int32_t)n;
  }
  if (bad) report(status, bad);
}

int launch_com(const int32_t* idx, const int64_t* off, int64_t frame0, int64_t n_frames,
               const stem_det& det, int64_t nplane, double* com64, float* com32, int32_t* counts,
               int32_t* status, hipStream_t stream) {
  if (n_frames == 0) return STEM_OK;
  const int ft = frame_threads(n_frames);
  const int64_t blocks = (n_frames + kComThreads / ft - 1) / (kComThreads / ft);
  STEM_TRACE("com_moments", stream);
  const PixDiv div = make_pixdiv(det.W, det.H, 1);
  const auto fn = ft == 4 ? (div.d24 ? k_com<true, 4> : k_com<false, 4>) : (div.d24 ? k_com<true, 2> : k_com<false, 2>);
  hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(kComThreads), 0, stream, idx, off, frame0, n_frames, div,
                     det.cx, det.cy, det.W * det.H, nplane, com64, com32, counts, status);
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

// ---------------------------------------------------------------------------------------------
// virtual annular detectors: the same split as k_com; a frame's threads count its events in each annulus
// [lo_j, hi_j) of squared pixel distance (exact int64 thresholds)
//
// D24 (sides below 2^15 and the zero-frequency pixel on the detector, so d^2 < 2^32): the squared distance by
// 24-bit multiplications and one unsigned comparison per annulus.

struct Annuli {
  int64_t lo[STEM_MAX_ANNULI], hi[STEM_MAX_ANNULI];
  uint32_t lo32[STEM_MAX_ANNULI], len32[STEM_MAX_ANNULI];  // lo and hi - lo, cut at 2^32 - 1
};

template <int NA, bool D24, int FT>
__global__ void __launch_bounds__(kComThreads) k_annular(const int32_t* __restrict__ idx,
                                                         const int64_t* __restrict__ off, int64_t frame0,
                                                         int64_t n_frames, PixDiv div, int32_t cx, int32_t cy,
                                                         int32_t npix, int32_t n_det, Annuli an, int64_t F,
                                                         int32_t* __restrict__ out, int32_t* status) {
  constexpr int kSumFrames = kComThreads / FT;
  __shared__ __align__(16) int32_t s_ev[kSumWin + 8];
  __shared__ int64_t s_off[kSumFrames + 1];
  const int f = threadIdx.x / FT, part = threadIdx.x % FT;
  const int64_t fb = frame0 + (int64_t)blockIdx.x * kSumFrames;
  const int64_t left = frame0 + n_frames - fb;
  const int nf = (int)(left < kSumFrames ? left : kSumFrames);
  if (!load_offsets(off, fb, nf, s_off, status)) return;
  const int64_t base = s_off[0];
  const int span = (int)(s_off[nf] - base);
  const int lo_f = f < nf ? (int)(s_off[f] - base) : 0, hi_f = f < nf ? (int)(s_off[f + 1] - base) : 0;
  int32_t cnt[NA];
#pragma unroll
  for (int j = 0; j < NA; ++j) cnt[j] = 0;
  uint32_t nbad = 0;
  for (int w0 = 0; w0 < span; w0 += kSumWin) {
    const int wn = span - w0 < kSumWin ? span - w0 : kSumWin;
    if (w0 > 0) __syncthreads();
    const int sh = stage_events<kSumWin>(idx, base + w0, wn, s_ev);
    __syncthreads();
    const int lo = (lo_f > w0 ? lo_f : w0) - w0 + sh;
    const int hi = (hi_f < w0 + wn ? hi_f : w0 + wn) - w0 + sh;
    frame_events<FT>(s_ev, lo, hi, part, [&](int32_t k) {
      const bool in = (uint32_t)k < (uint32_t)npix;
      nbad += in ? 0u : 1u;
      const uint32_t kk = in ? (uint32_t)k : 0u;
      const uint32_t ky = pix_row<D24>(kk, div), kx = pix_col<D24>(kk, ky, div);
      if constexpr (D24) {
        const int dx = (int)kx - cx, dy = (int)ky - cy;
        const uint32_t d2 = (uint32_t)__mul24(dx, dx) + (uint32_t)__mul24(dy, dy);
#pragma unroll
        for (int j = 0; j < NA; ++j) cnt[j] += (in && d2 - an.lo32[j] < an.len32[j]) ? 1 : 0;
      } else {
        const int64_t dx = (int64_t)kx - cx, dy = (int64_t)ky - cy;
        const int64_t d2 = dx * dx + dy * dy;
#pragma unroll
        for (int j = 0; j < NA; ++j) cnt[j] += (in && d2 >= an.lo[j] && d2 < an.hi[j]) ? 1 : 0;
      }
    });
  }
#pragma unroll
  for (int j = 0; j < NA; ++j) {
#pragma unroll
    for (int o = 1; o < FT; o <<= 1) cnt[j] += __shfl_xor(cnt[j], o);
    if (f < nf && part == 0 && j < n_det) out[(int64_t)j * F + fb + f] = cnt[j];  // NA is n_det rounded up
  }
  if (nbad) report(status, STEM_ERANGE);
}

// ---------------------------------------------------------------------------------------------
// sum of frames: the event range is split evenly over the workgroups; each counts its events into
// 32-bit LDS counters over a box of up to 128 x 128 pixels around the zero-frequency pixel, where
// the bright-field disk and nearly all events fall (events outside the box go straight to global
// atomics: kept in LDS until the box's turn they took 117 us in all, they overlap the events' loads here),
// then adds the box to the global sum once.
//
// Bound by those global atomics: every workgroup adds the whole disk.  So one large workgroup per compute unit
// (256 of 1024 threads), two counters per 64-bit atomic where the sum is aligned for it, and
// every workgroup starts its box at another place, so that they do not queue at the same lines.  Measured at 4.2e7 events in 2^20 frames (4% outside the disk): 165 us with 512 workgroups of
// 256 threads, 32-bit atomics and one order, 105 us now.

constexpr int kSumBox = 128;
constexpr int kSumBlocks = 256;
constexpr int kSumThreads = 1024;

template <bool D24, bool PAIR>
__global__ void __launch_bounds__(kSumThreads) k_sum_events(const int32_t* __restrict__ idx,
                                                            const int64_t* __restrict__ off, int64_t frame0,
                                                            int64_t n_frames, PixDiv div, int32_t npix, int32_t bx0,
                                                            int32_t by0, int32_t bw, int32_t bh,
                                                            uint32_t* __restrict__ sum, int32_t* status) {
  __shared__ __align__(8) uint32_t s_box[kSumBox * kSumBox];
  const int64_t e0 = off[frame0], e1 = off[frame0 + n_frames];
  if (e1 < e0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) report(status, STEM_EOFFSETS);
    return;
  }
  const int nbox = bw * bh;
  for (int i = threadIdx.x; i < nbox; i += kSumThreads) s_box[i] = 0u;
  __syncthreads();
  // this workgroup's share of the events, in whole 16-byte groups where possible
  const int64_t per = ((e1 - e0 + gridDim.x - 1) / gridDim.x + 3) & ~3ll;
  const int64_t a0 = e0 + (int64_t)blockIdx.x * per;
  const int64_t aend = a0 + per < e1 ? a0 + per : e1;
  uint32_t nbad = 0;
  if (a0 < aend) {
    const int sh = (int)((((uintptr_t)(idx + a0)) & 15) >> 2);
    const int64_t al = a0 - sh;
    const int64_t ng = (aend - al + 3) >> 2;
    auto add = [&](int32_t k, bool ok) {
      const bool in = ok && (uint32_t)k < (uint32_t)npix;
      nbad += ok && !in ? 1u : 0u;
      const uint32_t ky = pix_row<D24>((uint32_t)k, div);
      const int x = (int)pix_col<D24>((uint32_t)k, ky, div) - bx0, y = (int)ky - by0;
      const bool box = (uint32_t)x < (uint32_t)bw && (uint32_t)y < (uint32_t)bh;
      if (in && box) atomicAdd(&s_box[y * bw + x], 1u);
      else if (in) atomicAdd(&sum[k], 1u);
    };
    // whole 16-byte lines that hold at least one of the events (the others of the first and last line are
    // masked), U of them in flight per thread while the U before are counted
    constexpr int U = 4;
    int4 v[U];
    auto load = [&](int64_t g0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t g = g0 + u * kSumThreads;
        v[u] = *(const int4*)(idx + al + 4 * (g < ng ? g : ng - 1));
      }
    };
    load(threadIdx.x);
    for (int64_t g0 = threadIdx.x; g0 < ng; g0 += U * kSumThreads) {
      int4 c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) c[u] = v[u];
      load(g0 + U * kSumThreads);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t g = g0 + u * kSumThreads;
        if (g > 0 && g < ng - 1) {
          add(c[u].x, true);
          add(c[u].y, true);
          add(c[u].z, true);
          add(c[u].w, true);
        } else if (g < ng) {
          const int64_t e = al + 4 * g;
          add(c[u].x, e >= a0 && e < aend);
          add(c[u].y, e + 1 >= a0 && e + 1 < aend);
          add(c[u].z, e + 2 >= a0 && e + 2 < aend);
          add(c[u].w, e + 3 >= a0 && e + 3 < aend);
        }
      }
    }
  }
  __syncthreads();
  constexpr int P = PAIR ? 2 : 1;
  const int n = nbox / P, start = (int)((int64_t)n * blockIdx.x / gridDim.x);
  for (int i = threadIdx.x; i < n; i += kSumThreads) {
    const int p = P * (i + start < n ? i + start : i + start - n);
    uint32_t* dst = sum + (int64_t)(by0 + p / bw) * div.mg.d + bx0 + p % bw;
    if constexpr (PAIR) {
      // a left sum that wraps carries one into its neighbour, which is taken back (waiting for the old values
      // costs 0.8 us)
      const unsigned long long c = *(const unsigned long long*)&s_box[p];
      if (c) {
        const unsigned long long was = atomicAdd((unsigned long long*)dst, c);
        if ((uint32_t)was + (uint32_t)c < (uint32_t)c) atomicSub(dst + 1, 1u);
      }
    } else {
      const uint32_t c = s_box[p];
      if (c) atomicAdd(dst, c);
    }
  }
  if (nbad) report(status, STEM_ERANGE);
}

__global__ void __launch_bounds__(256) k_frame_mean(const uint32_t* __restrict__ sum, int64_t npix, double n,
                                                    float* __restrict__ mean) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < npix) mean[p] = (float)((double)sum[p] / n);
}

// ---------------------------------------------------------------------------------------------
// run-length form -> linear indices: the block's distances are staged in LDS like k_com's
// events, thread t replaces its frame's distances by their running sum in place, and the
// workgroup writes the window back with 16-byte stores (the store groups that are not wholly
// inside the window are written element by element).

__global__ void __launch_bounds__(kComThreads) k_decode_rle(const int32_t* __restrict__ dist,
                                                            const int64_t* __restrict__ off, int64_t frame0,
                                                            int64_t n_frames, int32_t npix,
                                                            int32_t* __restrict__ idx, int32_t* status) {
  __shared__ __align__(16) int32_t s_ev[kComWin + 8];
  __shared__ int32_t s_rel[kComFrames + 1];
  __shared__ int64_t s_base;
  const int t = threadIdx.x;
  const int64_t fb = frame0 + (int64_t)blockIdx.x * kComFrames;
  const int64_t left = frame0 + n_frames - fb;
  const int nf = (int)(left < kComFrames ? left : kComFrames);
  if (!load_rel_offsets(off, fb, nf, s_rel, &s_base, status)) return;
  __syncthreads();
  const int span = s_rel[nf];
  const int lo_t = t < nf ? s_rel[t] : 0, hi_t = t < nf ? s_rel[t + 1] : 0;
  int64_t run = 0;  // running sum of frame t, carried across windows
  uint32_t nbad = 0;
  for (int w0 = 0; w0 < span; w0 += kComWin) {
    const int wn = span - w0 < kComWin ? span - w0 : kComWin;
    __syncthreads();
    const int sh = stage_events<kComWin>(dist, s_base + w0, wn, s_ev);
    __syncthreads();
    const int lo = (lo_t > w0 ? lo_t : w0) - w0 + sh;
    const int hi = (hi_t < w0 + wn ? hi_t : w0 + wn) - w0 + sh;
    for (int e = lo; e < hi; ++e) {
      run += s_ev[e];
      const bool in = run >= 0 && run < npix;
      nbad += in ? 0u : 1u;
      s_ev[e] = in ? (int32_t)run : -1;
    }
    __syncthreads();
    // write back [sh, sh + wn) of the staging buffer to idx[s_base + w0 ...]
    const int64_t a0 = s_base + w0, aend = a0 + wn, al = a0 - sh;
    const int nchunk = (wn + sh + 3) >> 2;
    for (int c = t; c < nchunk; c += blockDim.x) {
      const int64_t e = al + 4 * (int64_t)c;
      if (e >= a0 && e + 4 <= aend && ((((uintptr_t)(idx + e)) & 15) == 0)) {
        *(int4*)(idx + e) = *(const int4*)&s_ev[4 * c];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (e + j >= a0 && e + j < aend) idx[e + j] = s_ev[4 * c + j];
      }
    }
  }
  if (nbad) report(status, STEM_ERANGE);
}

// ---------------------------------------------------------------------------------------------
// geometry of the kept set (one workgroup)

// The kept set's row runs and bin centres, by one workgroup of blockDim.x threads; s holds
// 3 * 1024 + 1 ints of LDS scratch.
__device__ void build_geometry(int32_t b, int32_t nbx, int32_t nby, int32_t cx, int32_t cy, double r2,
                               RowRun* __restrict__ rows, double2* __restrict__ kc, int32_t* s) {
  int32_t* s_lo = s;
  int32_t* s_hi = s + 1024;
  int32_t* s_start = s + 2048;
  int32_t& s_base = s[3072];
  if (threadIdx.x == 0) s_base = 0;
  // nby <= 4096 is checked on the host; rows are handled in slices of 1024
  for (int r0 = 0; r0 < nby; r0 += 1024) {
    const int nr = nby - r0 < 1024 ? nby - r0 : 1024;
    for (int r = threadIdx.x; r < nr; r += blockDim.x) {
      int lo, hi;
      kept_run(b, r0 + r, nbx, cx, cy, r2, lo, hi);
      s_lo[r] = lo;
      s_hi[r] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      int32_t base = s_base;
      for (int r = 0; r < nr; ++r) {
        s_start[r] = base;  // exclusive prefix of the run lengths
        base += s_hi[r] - s_lo[r];
      }
      s_base = base;
    }
    __syncthreads();
    for (int r = threadIdx.x; r < nr; r += blockDim.x) {
      RowRun rr;
      rr.start = s_start[r];
      rr.lo = s_lo[r];
      rr.hi = s_hi[r];
      rr.pad = 0;
      rows[r0 + r] = rr;
      const double ky = bin_centre(b, r0 + r, cy);
      for (int bx = rr.lo; bx < rr.hi; ++bx)
        kc[rr.start + bx - rr.lo] = make_double2(bin_centre(b, bx, cx), ky);
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(256) k_geometry(int32_t b, int32_t nbx, int32_t nby, int32_t cx,
                                                  int32_t cy, double r2, RowRun* __restrict__ rows,
                                                  double2* __restrict__ kc) {
  __shared__ int32_t s[3 * 1024 + 1];
  build_geometry(b, nbx, nby, cx, cy, r2, rows, kc, s);
}

// ---------------------------------------------------------------------------------------------
// pixel -> kept bin lookup: lut[ky*W + kx] = kd of the bin holding the pixel, -1 if that bin is
// dropped (its centre outside the disk)

__global__ void __launch_bounds__(256) k_pixel_lut(const RowRun* __restrict__ rows, int32_t W, int32_t H, int32_t b,
                                                   int16_t* __restrict__ lut) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (int64_t)W * H) return;
  const int ky = (int)(p / W), kx = (int)(p % W);
  const RowRun rr = rows[ky / b];
  const int bx = kx / b;
  lut[p] = (int16_t)(bx >= rr.lo && bx < rr.hi ? rr.start + bx - rr.lo : -1);
}

int launch_geometry(const stem_det& det, double r2, RowRun* rows, double2* kc, hipStream_t stream) {
  const int nbx = det.W / det.bin, nby = det.H / det.bin;
  STEM_TRACE("ssb_geometry", stream);
  hipLaunchKernelGGL(k_geometry, dim3(1), dim3(256), 0, stream, det.bin, nbx, nby, det.cx, det.cy, r2,
                     rows, kc);
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

// ---------------------------------------------------------------------------------------------
// binning into D[kd][f] (frames of whole scan rows)
//
// Workgroup = FR consecutive frames x a run of up to BinShape<FR>::kKd kept pixels (small workgroups:
// several per CU hide the latency of their load, count and write-out phases).  The block's events are
// streamed in windows of kBinWin: first threads write the frame numbers into an LDS byte map over the
// window's events, then the events are read with coalesced 16-byte loads (four per lane), their frames
// read from the map as one word and their pixels mapped by the lookup table.  Counts live in LDS: 8-bit counters, four frames per word, when every frame of the block has at
// most 255 events (no count can then carry into its neighbour); otherwise 16-bit counters, two frames
// per word, over two passes of half the pixels.  A count above the element type of D sets
// STEM_EOVERFLOW (the stored value is then not meaningful).
//
// FR = 128 writes whole 128-byte lines of D.  Where its counters do not hold all kept pixels, every chunk
// of pixels reads and looks up the block's events again: FR = 64 and 32 hold 351 and 800 pixels at
// once (bin_frames).

constexpr int kBinThreads = 256;
constexpr int kBinWin = 6144;       // events per window of the frame map (a block of 128 frames at 40
                                    // events per frame fits one)
constexpr int kBinBoxMax = 4096;    // bins of the largest LDS bin table (8 KB)

// Counters of a workgroup of FR frames: words of LDS (23 or 28 KB), and the pixels they hold.  Pixel rows
// of counters are FR/4 (+1 padding) words apart, so that the events of one frame (same column,
// different pixels) fall into different LDS banks.
template <int FR>
struct BinShape {
  static constexpr int kWords = FR == 32 ? 7200 : 5976;
  static constexpr int kKd = kWords / (FR / 4 + 1);  // 181, 351, 800
};

// The kept bins' bounding box (in bins) and the divisions that take a pixel to its bin: with it
// (BOX) the pixel -> bin table is a small per-workgroup LDS copy over the box, looked up with a
// division by W (magic number) and by the binning (multiply-high), instead of a gather from the
// global per-pixel table.
constexpr int kBoxRows = 64;  // bin rows of the largest box whose row runs travel as arguments
struct BinBox {
  PixDiv div;         // division by the detector width W and by the binning
  int32_t bin;
  int32_t bx0, by0, bw, bh;
  int32_t start[kBoxRows], lo[kBoxRows], hi[kBoxRows];  // row runs of the box's rows (BOX)
};

// The kept set's geometry, written by the first workgroup of the binning kernel (BOX)
struct GeomOut {
  RowRun* rows;       // nullptr: nothing to write
  double2* kc;
  int32_t nby, cx, cy;
  unsigned long long* mark;  // if set, cleared by the first thread (an accumulation from frame 0
                             // voids the state's FINALIZE)
};

// One step of a segmented inclusive scan within rows of 16 lanes: lane i adds the sums of lane
// i - d of its row when both hold the same key (sorted keys: equal keys are contiguous).  Lanes
// whose source lies before the row start get the sentinel key -1 and add nothing.
template <int CTRL>
__device__ __forceinline__ void seg_step(int key, int32_t& ax, int32_t& ay) {
  const int k2 = __builtin_amdgcn_update_dpp(-1, key, CTRL, 0xf, 0xf, false);
  const int x2 = __builtin_amdgcn_update_dpp(0, ax, CTRL, 0xf, 0xf, false);
  const int y2 = __builtin_amdgcn_update_dpp(0, ay, CTRL, 0xf, 0xf, false);
  if (k2 == key) {
    ax += x2;
    ay += y2;
  }
}

// With COM, the workgroups of the first pixel chunk also form each frame's exact integer first
// moments from the same event loads (Eq. 4): a lane folds its four events into runs of equal
// frame, a segmented scan over each row of 16 lanes (events are in frame order) merges the runs
// that cross lanes, and one LDS atomic per run end adds them to the frame's window sums (int32: a window
// holds at most kBinWin events, each |kx - cx| < 2^16), which thread f folds into its frame's
// int64 sums at the next window barrier.  The centre of mass is then S / N_f by one double
// division, as the centre-of-mass kernel computes it.
//
// BOX: the first nset workgroups bin nothing; the first writes the geometry, the others the interval table
// and the mask (with B >= 4 columns a set, one word per workgroup and every fourth column per wave, else
// one word per wave), beside the binning's rather than before it.
template <typename DT, bool BOX, bool COM, int FR, bool D24>
__global__ void __launch_bounds__(kBinThreads) k_bin(const int32_t* __restrict__ idx,
                                                     const int64_t* __restrict__ off, int64_t frame0,
                                                     int64_t n_frames, int32_t npix,
                                                     const int16_t* __restrict__ lut,
                                                     const RowRun* __restrict__ rows, BinBox box, int32_t n_k,
                                                     int64_t F, DT* __restrict__ D, ComOut com, GeomOut geo,
                                                     SetsJob sj, int nset, int64_t fblocks, int32_t* status) {
  constexpr int kKd = BinShape<FR>::kKd;
  extern __shared__ int16_t s_box[];  // [bh][bw] kept-bin index of each bin of the box, or -1
  __shared__ __align__(16) uint32_t s_hist[BinShape<FR>::kWords];
  __shared__ uint32_t s_map[(kBinWin + 16) / 4];
  // Relative to the block's first event, in 32 bits: with 64-bit offsets FR = 128 and its bin table passed the 32 KB
  // of five workgroups a compute unit from about 350 pixels on (1024 x 1024, 357 pixels: 227 instead of 199 us).
  __shared__ int32_t s_rel[FR + 1];
  __shared__ int32_t s_mom[COM ? 2 * FR : 1];  // [x | y][frame] moment sums of a window
  const int t = threadIdx.x;
  const int lane = t & 63;
  if (geo.mark && blockIdx.x == 0 && t == 0) *geo.mark = 0ull;
  if constexpr (BOX) {
    if ((int)blockIdx.x < nset) {
      // Kc of kept pixel kd from the box's row runs
      auto centre = [&](int kd) {
        int r = 0;
        while (r < box.bh - 1 && kd >= box.start[r] + box.hi[r] - box.lo[r]) ++r;
        return make_double2(bin_centre(box.bin, box.lo[r] + kd - box.start[r], geo.cx),
                            bin_centre(box.bin, box.by0 + r, geo.cy));
      };
      if (blockIdx.x == 0) {
        for (int r = t; r < geo.nby; r += kBinThreads) {
          const int q = r - box.by0;
          const bool in = q >= 0 && q < box.bh;
          geo.rows[r] = in ? RowRun{box.start[q], box.lo[q], box.hi[q], 0} : RowRun{q < 0 ? 0 : n_k, 0, 0, 0};
        }
        for (int kd = t; kd < n_k; kd += kBinThreads) geo.kc[kd] = centre(kd);
        return;
      }
      const int w = t >> 6;
      const bool split = sj.B >= 4;
      const int64_t word = split ? (int64_t)blockIdx.x - 1 : (int64_t)(blockIdx.x - 1) * (kBinThreads / 64) + w;
      const bool live = word < (int64_t)sj.ncs * sj.nmw;  // the same for the whole wave
      uint64_t bits = 0;
      if (live) {
        const int kd = 64 * (int)(word % sj.nmw) + lane;
        const double2 k = kd < sj.n_k ? centre(kd) : make_double2(0.0, 0.0);
        bits = sets_columns(sj, word, lane, k, split ? w : 0, split ? 4 : 1);
      }
      if (split) {
        uint64_t* s_bits = (uint64_t*)s_hist;
        if (lane == 0) s_bits[w] = bits;
        __syncthreads();
        bits = s_bits[0] | s_bits[1] | s_bits[2] | s_bits[3];
        if (t == 0 && live) sj.mask[word] = bits;
      } else if (lane == 0 && live) {
        sj.mask[word] = bits;
      }
      return;
    }
  }
  const int nchunks = (n_k + kKd - 1) / kKd;
  const int64_t blk = (int64_t)blockIdx.x - nset;
  const int kd0 = (int)(blk % nchunks) * kKd;
  const int kc = n_k - kd0 < kKd ? n_k - kd0 : kKd;
  int64_t fblk = blk / nchunks;
  // Blocks of less than 128 frames share D's 128-byte lines with their neighbours: consecutive ones go to
  // the same XCD (workgroups go round the 8 of them), whose L2 then joins the parts of a line.
  if (FR < 128 && nchunks == 1 && (fblocks & 7) == 0) fblk = (fblk & 7) * (fblocks >> 3) + (fblk >> 3);
  const int64_t fb = frame0 + fblk * FR;
  const int64_t fend = frame0 + n_frames;
  const int nf = (int)((fend - fb) < FR ? (fend - fb) : FR);
  const int64_t base = off[fb], events = off[fb + nf] - base;
  if (events >= (1ll << 30)) {  // the 32-bit relative offsets cannot address that many events
    if (t == 0) report(status, STEM_EOVERFLOW);
    return;
  }
  const int span = (int)events;
  if (t <= nf) s_rel[t] = (int32_t)(off[fb + t] - base);
  const bool com_blk = COM && kd0 == 0;  // workgroup-uniform
  if constexpr (COM) {
    if (com_blk)
      for (int i = t; i < 2 * FR; i += kBinThreads) s_mom[i] = 0;
  }
  int64_t msx = 0, msy = 0;  // thread t: the moments of frame t so far
  // after a barrier that follows a window's atomics and precedes the next window's
  auto fold_moments = [&]() {
    if (COM && com_blk && t < FR) {
      msx += s_mom[t];
      msy += s_mom[FR + t];
      s_mom[t] = 0;
      s_mom[FR + t] = 0;
    }
  };
  __syncthreads();
  if constexpr (BOX) {
    // kept index of each bin of the box from the row runs (the rule of the per-pixel table)
    for (int i = t; i < box.bw * box.bh; i += kBinThreads) {
      const int ry = i / box.bw, bx = box.bx0 + i % box.bw;
      s_box[i] = (int16_t)(bx >= box.lo[ry] && bx < box.hi[ry] ? box.start[ry] + bx - box.lo[ry] : -1);
    }
  }
  const int wide = __syncthreads_or(t < nf && s_rel[t + 1] - s_rel[t] > 255);
  // the frame whose map entries this thread writes, and its part of them among the S threads of the frame, each
  // a run of whole words.  (The S threads beside each other, every S-th word each with both ends tested: FR = 128
  // took 198 instead of 188 us at 1024 x 1024 with 357 pixels, 624 instead of 527 us at 256 x 256 with 707 and
  // 400 events a frame; one thread a frame 191 and 582 us.)
  constexpr int S = kBinThreads / FR;
  const int mf = t % FR, mp = t / FR;
  const int lo_m = mf < nf ? s_rel[mf] : 0, hi_m = mf < nf ? s_rel[mf + 1] : 0;
  uint8_t* map = (uint8_t*)s_map;
  int32_t bad = 0;
  const int npass = wide ? 2 : 1;
  const int kpp = (kc + npass - 1) / npass;       // pixels per pass
  const int wpr = wide ? FR / 2 : FR / 4;         // words per pixel row
  const int wps = wpr + 1;                        // row stride in words (padded)
  const uint32_t cap = sizeof(DT) == 1 ? 255u : 65535u;
  // 8-bit counts go out as 16 frames (four counter words) per 16-byte store, 16-bit ones as 4 frames (one
  // word) per 8-byte store, when aligned
  const bool vec = !wide && (((uintptr_t)D & 15) == 0) &&
                   (sizeof(DT) == 1 ? (F & 15) == 0 && (fb & 15) == 0 : (F & 3) == 0 && (fb & 3) == 0);
  for (int pass = 0; pass < npass; ++pass) {
    const int ka = kd0 + pass * kpp;
    const int kn = (kd0 + kc) - ka < kpp ? (kd0 + kc) - ka : kpp;
    for (int i = t; i < (kn * wps + 3) >> 2; i += kBinThreads) ((uint4*)s_hist)[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int w0 = 0; w0 < span; w0 += kBinWin) {
      const int wn = span - w0 < kBinWin ? span - w0 : kBinWin;
      const int64_t a0 = base + w0;
      const int sh = (int)((((uintptr_t)(idx + a0)) & 15) >> 2);  // map[sh + j] <-> event a0 + j
      if (w0 > 0) {
        __syncthreads();
        fold_moments();
      }
      {
        // frame mf's events of this window: map entries [lo, hi), of which this thread's part
        const int lo = (lo_m > w0 ? lo_m : w0) - w0 + sh;
        const int hi = (hi_m < w0 + wn ? hi_m : w0 + wn) - w0 + sh;
        const uint32_t word = (uint32_t)mf * 0x01010101u;
        auto cut = [&](int m) { return m == 0 ? lo : m == S ? hi : min((lo + (hi - lo) * m / S + 3) & ~3, hi); };
        if (lo < hi) {
          const int end = cut(mp + 1);
          int j = cut(mp);
          for (; j < end && (j & 3); ++j) map[j] = (uint8_t)mf;
          for (; j + 4 <= end; j += 4) s_map[j >> 2] = word;
          for (; j < end; ++j) map[j] = (uint8_t)mf;
        }
      }
      __syncthreads();
      // Positions p = 4 g + q of the 16-byte aligned run from ib: [sh, sh + wn) are this window's
      // events.  Every group g < ng holds at least one of them, so its whole 16-byte line lies in
      // the event array's pages; the other positions of the line are masked out.  (Loaded before the
      // map is written, the events cost 12 registers and a wave per SIMD: 121 against 104 us at
      // 1024 x 1024, 59 against 52 us at 512 x 512 binned 6x.)
      const int32_t* ib = idx + (a0 - sh);
      const int ng = (wn + sh + 3) >> 2;
      constexpr int U = kBinWin / (4 * kBinThreads);  // groups per thread in flight: one trip per window (a
                                                      // full one off a 16-byte line has a group more)
      for (int g0 = t; g0 < ng; g0 += U * kBinThreads) {
        int4 kv[U];
        uint32_t fr4[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int g = g0 + u * kBinThreads;
          kv[u] = make_int4(0, 0, 0, 0);
          fr4[u] = 0u;
          if (g < ng) {
            kv[u] = *(const int4*)(ib + 4 * g);
            fr4[u] = s_map[g];
          }
        }
        // the table lookups are issued together; masked or out-of-range positions look up pixel 0
        int kd[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int p = 4 * (g0 + u * kBinThreads) + q;
            const int k = q == 0 ? kv[u].x : q == 1 ? kv[u].y : q == 2 ? kv[u].z : kv[u].w;
            const bool ok = (uint32_t)(p - sh) < (uint32_t)wn;
            const bool in = (uint32_t)k < (uint32_t)npix;
            if (ok && !in) bad |= STEM_ERANGE;
            const uint32_t kk = ok && in ? (uint32_t)k : 0u;  // 32-bit offset from the table base
            int v;
            if constexpr (BOX) {
              const uint32_t ky = pix_row<D24>(kk, box.div), kx = pix_col<D24>(kk, ky, box.div);
              const uint32_t rx = pix_bin<D24>(kx, box.div) - (uint32_t)box.bx0;
              const uint32_t ry = pix_bin<D24>(ky, box.div) - (uint32_t)box.by0;
              v = rx < (uint32_t)box.bw && ry < (uint32_t)box.bh ? (int)s_box[ry * box.bw + rx] : -1;
            } else {
              v = (int)*(const int16_t*)((const char*)lut + 2u * kk);
            }
            kd[u][q] = ok && in && v >= 0 ? v - ka : -1;
          }
        if constexpr (COM) {
          if (com_blk && pass == 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
              // runs of equal frame among the lane's events in this window; all but the last go
              // to LDS at once (a lane crosses a frame boundary only at frames of few events)
              int fc = -1;
              int32_t ax = 0, ay = 0;
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const int p = 4 * (g0 + u * kBinThreads) + q;
                if ((uint32_t)(p - sh) >= (uint32_t)wn) continue;
                const int k = q == 0 ? kv[u].x : q == 1 ? kv[u].y : q == 2 ? kv[u].z : kv[u].w;
                const int f = (int)((fr4[u] >> (8 * q)) & 0xffu);
                if (f != fc) {
                  if (fc >= 0) {
                    atomicAdd(&s_mom[fc], ax);
                    atomicAdd(&s_mom[FR + fc], ay);
                  }
                  fc = f;
                  ax = ay = 0;
                }
                // an index outside the detector adds nothing (it is reported by the binning)
                if ((uint32_t)k < (uint32_t)npix) {
                  const uint32_t ky = pix_row<D24>((uint32_t)k, box.div), kx = pix_col<D24>((uint32_t)k, ky, box.div);
                  ax += (int32_t)kx - com.cx;
                  ay += (int32_t)ky - com.cy;
                }
              }
              // the lanes' last runs: inclusive scan within each row of 16 lanes, segmented by
              // frame, by DPP row shifts (register moves, no LDS traffic); lower lanes hold
              // earlier events, and the lanes of this loop trip are a prefix of the wave
              const int key = fc >= 0 ? fc : 256 + lane;  // a lane without events merges with none
              seg_step<0x111>(key, ax, ay);               // row_shr:1
              seg_step<0x112>(key, ax, ay);               // row_shr:2
              seg_step<0x114>(key, ax, ay);               // row_shr:4
              seg_step<0x118>(key, ax, ay);               // row_shr:8
              // a run ends where the next lane's frame differs, at a row's last lane (row_shl:1
              // leaves the sentinel there) and before a lane outside this loop trip
              const int nkey = __builtin_amdgcn_update_dpp(-2, key, 0x101, 0xf, 0xf, false);
              const bool last = g0 + 1 >= ng || nkey != key;
              if (fc >= 0 && last) {
                atomicAdd(&s_mom[fc], ax);
                atomicAdd(&s_mom[FR + fc], ay);
              }
            }
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            // a dropped bin (-1), or a pixel of another chunk or pass, is not counted here
            if ((uint32_t)kd[u][q] >= (uint32_t)kn) continue;
            const uint32_t f = (fr4[u] >> (8 * q)) & 0xffu;
            const int shift = wide ? 16 * (f & 1) : 8 * (f & 3);
            const int col = wide ? (f >> 1) : (f >> 2);
            atomicAdd(&s_hist[__umul24(kd[u][q], wps) + col], 1u << shift);
          }
      }
    }
    __syncthreads();
    if (vec && sizeof(DT) == 2) {
      // one counter word (4 frames) of one pixel row per thread and step
      for (int i = t; i < kn * wpr; i += kBinThreads) {
        const int kd = i / wpr, q = i % wpr;
        const int f0 = 4 * q;
        if (f0 >= nf) continue;
        const uint32_t w = s_hist[kd * wps + q];
        DT* dst = D + (int64_t)(ka + kd) * F + (fb + f0);
        if (f0 + 4 <= nf)
          *(uint2*)dst = make_uint2((w & 0xffu) | ((w & 0xff00u) << 8), ((w >> 16) & 0xffu) | ((w >> 24) << 16));
        else
          for (int j = 0; f0 + j < nf; ++j) dst[j] = (DT)((w >> (8 * j)) & 0xffu);
      }
    } else if (vec) {
      // four counter words (16 frames) of one pixel row per thread and step
      const int qpr = wpr / 4;
      for (int i = t; i < kn * qpr; i += kBinThreads) {
        const int kd = i / qpr, q4 = i % qpr;
        const int f0 = 16 * q4;
        if (f0 >= nf) continue;
        const uint32_t* hw = s_hist + kd * wps + 4 * q4;
        uint8_t* dst = (uint8_t*)D + (int64_t)(ka + kd) * F + (fb + f0);
        if (f0 + 16 <= nf) {
          *(uint4*)dst = make_uint4(hw[0], hw[1], hw[2], hw[3]);
        } else {
          for (int j = 0; f0 + j < nf; ++j) dst[j] = (uint8_t)(hw[j >> 2] >> (8 * (j & 3)));
        }
      }
    } else {
      // one counter word per thread and step: fpw consecutive frames of one pixel row
      const int fpw = wide ? 2 : 4;
      for (int i = t; i < kn * wpr; i += kBinThreads) {
        const int kd = i / wpr, q = i % wpr;
        const int f0 = q * fpw;
        if (f0 >= nf) continue;
        const uint32_t w = s_hist[kd * wps + q];
        uint32_t c[4];
        if (wide) {
          c[0] = w & 0xffffu;
          c[1] = w >> 16;
          c[2] = c[3] = 0u;
        } else {
          c[0] = w & 0xffu;
          c[1] = (w >> 8) & 0xffu;
          c[2] = (w >> 16) & 0xffu;
          c[3] = w >> 24;
        }
        DT* dst = D + (int64_t)(ka + kd) * F + (fb + f0);
        for (int j = 0; j < fpw && f0 + j < nf; ++j) {
          if (c[j] > cap) bad |= STEM_EOVERFLOW;
          dst[j] = (DT)c[j];
        }
      }
    }
    __syncthreads();
  }
  if constexpr (COM) {
    fold_moments();  // the pass loop ends with a barrier: the last window's sums
    if (com_blk && t < nf) {
      const int64_t fr = fb + t;
      const int64_t n = s_rel[t + 1] - s_rel[t];
      const int64_t sx = msx, sy = msy;
      const double x = n > 0 ? (double)sx / (double)n : 0.0;
      const double y = n > 0 ? (double)sy / (double)n : 0.0;
      if (com.com64) {
        com.com64[fr] = x;
        com.com64[com.nplane + fr] = y;
      }
      if (com.com32) {
        com.com32[fr] = (float)x;
        com.com32[com.nplane + fr] = (float)y;
      }
      if (com.counts) com.counts[fr] = (int32_t)n;
    }
  }
  if (bad) report(status, bad);
}

// The kept bins' bounding box and its rows' runs; true when the binning uses the LDS bin table
// over it (and then also takes the geometry's and the interval table's work).
static bool make_box(const stem_det& det, double r2, BinBox& box) {
  const int nbx = det.W / det.bin, nby = det.H / det.bin;
  box = BinBox{};
  int bxa = nbx, bxb = 0, bya = nby, byb = 0;
  int run_start = 0;
  for (int by = 0; by < nby; ++by) {
    int lo, hi;
    kept_run(det.bin, by, nbx, det.cx, det.cy, r2, lo, hi);
    if (hi <= lo) continue;
    bxa = lo < bxa ? lo : bxa;
    bxb = hi > bxb ? hi : bxb;
    if (bya == nby) bya = by;
    byb = by + 1;
    // row runs of the box's rows, in box-row order (kept rows of the box are contiguous)
    if (by - bya < kBoxRows) {
      box.start[by - bya] = run_start;
      box.lo[by - bya] = lo;
      box.hi[by - bya] = hi;
    }
    run_start += hi - lo;
  }
  box.bin = det.bin;
  box.div = make_pixdiv(det.W, det.H, det.bin);
  box.bx0 = bxa;
  box.by0 = bya;
  box.bw = bxb > bxa ? bxb - bxa : 0;
  box.bh = byb > bya ? byb - bya : 0;
  // the LDS table when it is small; the bin divisions by multiply-high are exact for W, H < 2^16
  const int64_t cells = (int64_t)box.bw * box.bh;
  return cells > 0 && cells <= kBinBoxMax && box.bh <= kBoxRows && det.W < 65536 && det.H < 65536;
}

// Frames per workgroup for n_k pixels.  A workgroup costs 8 to 10 us before its events count (tables, map, the
// chain of loads and LDS phases): where there are more of them than the GPU holds, 64 and 32 frames take 1.5 and 3
// times as long a chunk of pixels as 128.  They gain where they take fewer chunks (every chunk looks every event up
// again), the more events a frame the more (past 48 a workgroup of 128 frames takes a second window of kBinWin),
// or where the GPU is not full.  The host does not know the events a frame, so the lines lie where the smaller
// workgroup is not slower at 10 to 45 of them either.  One MI355X, 576 x 576 detector, us with FR = 128 / 64 / 32 at
// 10 events a frame, then at 100 (1024 x 1024: at 45):
//  - to 181 pixels, one chunk with any FR: 176 pixels, 1024 x 1024 frames 77 / 124 / 255, 102 / 155 / 299.
//  - to 351, one chunk from 64 down: 345 pixels, 512 x 512 frames 46 / 45 / 79, 128 / 84 / 89; 1024 x 1024 173 / 176 /
//    310, 192 / 186 / 337.
//  - to 800, one chunk of 32 against c of 128: up to 2^15 frames for c = 2, 2^16 for 3, 2^18 for 4, any number for 5.
//    370 pixels (3), 64 x 512 frames 18 / 19 / 21, 40 / 30 / 23; 512 x 512 60 / 74 / 79, 174 / 145 / 89.  707 (4), 512 x 512
//    95 / 125 / 92, 265 / 244 / 131; 1024 x 1024 412 / 585 / 459, 436 / 590 / 467.  790 (5), 1024 x 1024 (10; 40 events)
//    515 / 614 / 498, 577 / 660 / 519.
//  - more, several chunks of any: 32 up to 2^13 frames, 64 up to 2^16.  900 pixels, 64 x 64 frames 20 / 21 / 20, 33 / 24 /
//    19; 64 x 512 29 / 30 / 39, 67 / 50 / 40; 512 x 512 118 / 132 / 208, 332 / 259 / 223; 1024 x 1024 522 / 632 / 898, 563 /
//    653 / 920.
int bin_frames(int n_k, int64_t n_frames) {
  constexpr int k128 = BinShape<128>::kKd, k64 = BinShape<64>::kKd, k32 = BinShape<32>::kKd;
  if (n_k <= k128) return 128;
  if (n_k <= k64) return 64;
  if (n_k <= k32) {
    const int c = (n_k + k128 - 1) / k128;
    return c >= 5 || n_frames <= (c == 2 ? 1 << 15 : c == 3 ? 1 << 16 : 1 << 18) ? 32 : 128;
  }
  return n_frames <= 1 << 13 ? 32 : n_frames <= 1 << 16 ? 64 : 128;
}

bool bin_builds_sets(const stem_det& det, double r2) {
  BinBox box;
  return make_box(det, r2, box);
}

int launch_bin(const int32_t* idx, const int64_t* off, int64_t frame0, int64_t n_frames,
               const stem_det& det, double r2, RowRun* rows, double2* kc, int16_t* lut, int n_k, int64_t F,
               void* D, int d_bits, int32_t* status, hipStream_t stream, const ComOut* com, const SetsJob* sets,
               unsigned long long* mark) {
  if (n_frames == 0) return STEM_OK;
  BinBox box;
  const bool use_box = make_box(det, r2, box);
  const int64_t cells = (int64_t)box.bw * box.bh;
  const size_t lds = use_box ? (size_t)((cells * 2 + 15) & ~15ll) : 0;
  // BOX: a workgroup for the geometry and those of the interval table, a multiple of 8 (the rest follow in
  // the order of the XCDs)
  const SetsJob sj = use_box && sets ? *sets : SetsJob{};
  int nset = 0;
  if (use_box) {
    const int64_t words = sj.cst ? (int64_t)sj.ncs * sj.nmw : 0;
    nset = (int)((1 + (sj.B >= 4 ? words : (words + kBinThreads / 64 - 1) / (kBinThreads / 64)) + 7) & ~7ll);
  }
  const int fr = bin_frames(n_k, n_frames);
  const int kd = fr == 128 ? BinShape<128>::kKd : fr == 64 ? BinShape<64>::kKd : BinShape<32>::kKd;
  const int64_t fblocks = (n_frames + fr - 1) / fr;
  const dim3 grid((unsigned)(nset + fblocks * ((n_k + kd - 1) / kd)));
  // BOX: the binning kernel's first workgroup writes the row runs and bin centres; otherwise the
  // per-pixel table needs them first
  GeomOut geo{};
  if (use_box) {
    geo = GeomOut{rows, kc, det.H / det.bin, det.cx, det.cy, nullptr};
  } else {
    if (int st = launch_geometry(det, r2, rows, kc, stream)) return st;
    // the per-pixel table, read by the binning kernel
    STEM_TRACE("pixel_lut", stream);
    const int64_t npix = (int64_t)det.W * det.H;
    hipLaunchKernelGGL(k_pixel_lut, dim3((unsigned)((npix + 255) / 256)), dim3(256), 0, stream, rows, det.W, det.H,
                       det.bin, lut);
    STEM_LAUNCH_CHECK();
  }
  geo.mark = mark;
  STEM_TRACE(com ? "bin_com" : "bin_densify", stream);
  const ComOut co = com ? *com : ComOut{};
  const int npix = det.W * det.H;
  auto launch = [&](auto dt, auto bx, auto cm, auto frames) {
    using DT = decltype(dt);
    constexpr bool BX = decltype(bx)::value, CM = decltype(cm)::value;
    constexpr int FR = decltype(frames)::value;
    const auto fn = box.div.d24 ? k_bin<DT, BX, CM, FR, true> : k_bin<DT, BX, CM, FR, false>;
    hipLaunchKernelGGL(fn, grid, dim3(kBinThreads), BX ? lds : 0, stream, idx, off, frame0, n_frames, npix, lut, rows,
                       box, n_k, F, (DT*)D, co, geo, sj, nset, fblocks, status);
  };
  auto go = [&](auto dt, auto bx, auto cm) {
    if (fr == 128) launch(dt, bx, cm, std::integral_constant<int, 128>{});
    else if (fr == 64) launch(dt, bx, cm, std::integral_constant<int, 64>{});
    else launch(dt, bx, cm, std::integral_constant<int, 32>{});
  };
  using T_ = std::true_type;
  using F_ = std::false_type;
  if (d_bits == 8) {
    if (use_box) com ? go(uint8_t{}, T_{}, T_{}) : go(uint8_t{}, T_{}, F_{});
    else com ? go(uint8_t{}, F_{}, T_{}) : go(uint8_t{}, F_{}, F_{});
  } else {
    if (use_box) com ? go(uint16_t{}, T_{}, T_{}) : go(uint16_t{}, T_{}, F_{});
    else com ? go(uint16_t{}, F_{}, T_{}) : go(uint16_t{}, F_{}, F_{});
  }
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

}  // namespace stem

// ---------------------------------------------------------------------------------------------
// C ABI

using namespace stem;

extern "C" const char* stem_strerror(int status) {
  switch (status) {
    case STEM_OK: return "ok";
    case STEM_EINVAL: return "invalid argument";
    case STEM_ERANGE: return "event index outside the detector";
    case STEM_EOFFSETS: return "frame offsets not monotone or inconsistent with the event count";
    case STEM_EOVERFLOW: return "binned count does not fit the element type";
    case STEM_EWORKSPACE: return "workspace or state buffer too small or misaligned";
    case STEM_EHIP: return "HIP runtime error";
    case STEM_ESTATE: return "state buffer not prepared for this mode";
    default: return "several errors (status bits)";
  }
}

extern "C" int stem_version(void) { return 100; }

extern "C" int eer_load_csr(const int32_t* h_idx, const int64_t* h_off, int64_t frame0,
                            int64_t n_frames, int64_t n_events, const stem_det* det, int32_t* d_idx,
                            int64_t* d_off, int32_t* d_status, void* stream_) {
  if (!det || !d_idx || !d_off || frame0 < 0 || n_frames < 0 || n_events < 0) return STEM_EINVAL;
  if (det->W <= 0 || det->H <= 0 || (int64_t)det->W * det->H >= (1ll << 31)) return STEM_EINVAL;
  if ((h_idx == nullptr) != (h_off == nullptr)) return STEM_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  if (h_off) {
    if (h_off[0] < 0 || h_off[n_frames] - h_off[0] != n_events) return STEM_EINVAL;
    STEM_HIP_CHECK(hipMemcpyAsync(d_off + frame0, h_off, sizeof(int64_t) * (n_frames + 1),
                                  hipMemcpyHostToDevice, stream));
    if (n_events > 0)
      STEM_HIP_CHECK(hipMemcpyAsync(d_idx + h_off[0], h_idx, sizeof(int32_t) * n_events,
                                    hipMemcpyHostToDevice, stream));
  }
  // copy mode: the chunk's events occupy exactly [h_off[0], h_off[0] + n_events);
  // validate-only mode: d_idx holds n_events entries and the chunk must lie inside them
  const int64_t lo = h_off ? h_off[0] : 0;
  const int64_t hi = h_off ? h_off[0] + n_events : n_events;
  int64_t work = n_frames > n_events ? n_frames : n_events;
  int64_t blocks = (work + 255) / 256;
  if (blocks < 1) blocks = 1;
  if (blocks > 4096) blocks = 4096;
  {
    STEM_TRACE("csr_validate", stream);
    hipLaunchKernelGGL(k_validate, dim3((unsigned)blocks), dim3(256), 0, stream, d_idx, d_off, frame0,
                       n_frames, n_events, h_off ? 1 : 0, lo, hi, det->W * det->H, d_status);
  }
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

extern "C" int virtual_annular(const int32_t* d_idx, const int64_t* d_off, int64_t frame0, int64_t n_frames,
                               const stem_det* det, const stem_scan* scan, int n_det, const double* h_r_in,
                               const double* h_r_out, int32_t* d_out, int32_t* d_status, void* stream_) {
  if (!d_idx || !d_off || !det || !scan || !d_out || !h_r_in || !h_r_out) return STEM_EINVAL;
  if (det->W <= 0 || det->H <= 0 || (int64_t)det->W * det->H >= (1ll << 31)) return STEM_EINVAL;
  if (scan->ny <= 0 || scan->nx <= 0 || n_det < 1 || n_det > STEM_MAX_ANNULI) return STEM_EINVAL;
  const int64_t F = (int64_t)scan->ny * scan->nx;
  if (frame0 < 0 || n_frames < 0 || frame0 + n_frames > F) return STEM_EINVAL;
  Annuli an;
  const double big = 9.0e18;  // beyond every squared distance of a detector with W*H < 2^31
  for (int j = 0; j < STEM_MAX_ANNULI; ++j) {
    an.lo[j] = an.hi[j] = 0;
    if (j >= n_det) continue;
    const double a = h_r_in[j], b = h_r_out[j];
    if (!(a >= 0.0) || !(b >= 0.0)) return STEM_EINVAL;  // also rejects NaN
    // d2 >= a^2 and d2 < b^2 for an integer d2  <=>  d2 >= ceil(a^2) and d2 < ceil(b^2)
    const double a2 = std::ceil(a * a), b2 = std::ceil(b * b);
    an.lo[j] = a2 >= big ? (int64_t)big : (int64_t)a2;
    an.hi[j] = b2 >= big ? (int64_t)big : (int64_t)b2;
  }
  if (n_frames == 0) return STEM_OK;
  hipStream_t s = (hipStream_t)stream_;
  const int ft = frame_threads(n_frames);
  const int64_t blocks = (n_frames + kComThreads / ft - 1) / (kComThreads / ft);
  for (int j = 0; j < STEM_MAX_ANNULI; ++j) {
    const int64_t top = 0xffffffffll, lo = an.lo[j] < top ? an.lo[j] : top, hi = an.hi[j] < top ? an.hi[j] : top;
    an.lo32[j] = (uint32_t)lo;
    an.len32[j] = hi > lo ? (uint32_t)(hi - lo) : 0u;
  }
  const PixDiv div = make_pixdiv(det->W, det->H, 1);
  const bool d24 = div.d24 && det->cx >= 0 && det->cx <= det->W && det->cy >= 0 && det->cy <= det->H;
  STEM_TRACE("virtual_annular", s);
  const dim3 grid((unsigned)blocks), blk(kComThreads);
  const int npix = det->W * det->H;
  auto go = [&](auto na) {
    constexpr int NA = decltype(na)::value;
    const auto fn = ft == 4 ? (d24 ? k_annular<NA, true, 4> : k_annular<NA, false, 4>)
                            : (d24 ? k_annular<NA, true, 2> : k_annular<NA, false, 2>);
    hipLaunchKernelGGL(fn, grid, blk, 0, s, d_idx, d_off, frame0, n_frames, div, det->cx, det->cy, npix, n_det, an, F,
                       d_out, d_status);
  };
  if (n_det <= 1) go(std::integral_constant<int, 1>{});
  else if (n_det <= 2) go(std::integral_constant<int, 2>{});
  else if (n_det <= 4) go(std::integral_constant<int, 4>{});
  else if (n_det <= 8) go(std::integral_constant<int, 8>{});
  else go(std::integral_constant<int, 16>{});
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

extern "C" int sum_frames(const int32_t* d_idx, const int64_t* d_off, int64_t frame0, int64_t n_frames,
                          const stem_det* det, uint32_t* d_sum, float* d_mean, int32_t* d_status, void* stream_) {
  if (!d_idx || !d_off || !det || !d_sum || frame0 < 0 || n_frames <= 0) return STEM_EINVAL;
  if (det->W <= 0 || det->H <= 0 || (int64_t)det->W * det->H >= (1ll << 31)) return STEM_EINVAL;
  hipStream_t s = (hipStream_t)stream_;
  const int W = det->W, H = det->H;
  const int bw = W < kSumBox ? W : kSumBox, bh = H < kSumBox ? H : kSumBox;
  int bx0 = det->cx - bw / 2, by0 = det->cy - bh / 2;
  bx0 = bx0 < 0 ? 0 : (bx0 > W - bw ? W - bw : bx0);
  by0 = by0 < 0 ? 0 : (by0 > H - bh ? H - bh : by0);
  {
    STEM_TRACE("sum_frames", s);
    const PixDiv div = make_pixdiv(W, H, 1);
    // pairs of counters: even rows of the sum and of the box, from an 8-byte boundary
    const bool pair = ((uintptr_t)d_sum & 7) == 0 && W % 2 == 0 && bx0 % 2 == 0 && bw % 2 == 0;
    const auto fn = div.d24 ? (pair ? k_sum_events<true, true> : k_sum_events<true, false>)
                            : (pair ? k_sum_events<false, true> : k_sum_events<false, false>);
    hipLaunchKernelGGL(fn, dim3(kSumBlocks), dim3(kSumThreads), 0, s, d_idx, d_off, frame0, n_frames, div, W * H, bx0,
                       by0, bw, bh, d_sum, d_status);
    STEM_LAUNCH_CHECK();
  }
  if (d_mean) {
    const int64_t npix = (int64_t)W * H;
    hipLaunchKernelGGL(k_frame_mean, dim3((unsigned)((npix + 255) / 256)), dim3(256), 0, s, d_sum, npix,
                       (double)n_frames, d_mean);
    STEM_LAUNCH_CHECK();
  }
  return STEM_OK;
}

extern "C" int eer_decode_rle(const int32_t* d_dist, const int64_t* d_off, int64_t frame0, int64_t n_frames,
                              const stem_det* det, int32_t* d_idx, int32_t* d_status, void* stream_) {
  if (!d_dist || !d_off || !det || !d_idx || frame0 < 0 || n_frames < 0) return STEM_EINVAL;
  if (det->W <= 0 || det->H <= 0 || (int64_t)det->W * det->H >= (1ll << 31)) return STEM_EINVAL;
  if (n_frames == 0) return STEM_OK;
  hipStream_t s = (hipStream_t)stream_;
  const int64_t blocks = (n_frames + kComFrames - 1) / kComFrames;
  STEM_TRACE("decode_rle", s);
  hipLaunchKernelGGL(k_decode_rle, dim3((unsigned)blocks), dim3(kComThreads), 0, s, d_dist, d_off, frame0, n_frames,
                     det->W * det->H, d_idx, d_status);
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

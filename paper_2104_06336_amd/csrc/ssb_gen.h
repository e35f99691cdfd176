// Column transform fused with Eq. 3 at any scan length (fft_generic.h): the sum of the scans whose
// sides the wavefront kernels of ssb_fused.h do not both take.
//
// A workgroup owns one half-spectrum column c and a group of kept pixels.  It takes RB pixels at a time:
// their row-transformed columns X[kd][c][0..Ny) are transformed together as the rows of one LDS
// buffer, and G never leaves the chip: the last pass keeps its outputs in registers, where thread t
// holds the frequencies my = j + q Ny/R (q < R) of pixel slot t / (Ny/R), the same for every pixel, so
// the sums of T over the pixels are registers as well (acc, for the column itself and for its mirror
// Nx - c with conj G).  At the end the RB slots are added through LDS, in order.  Only pixels with a
// pair in the column or its mirror are read.  The columns of the next RB pixels are loaded while these
// are transformed.  With PWRITE the double-overlap values are also stored (the pruned array of
// ssb_fused.h).
//
// Bound by the transform's LDS traffic and arithmetic, as the fused sum of the fast lengths.  Measured
// (one MI355X, without aberrations): 1000 x 1000 scan, 176 pixels, storing the values, 505 us against
// 1620 us for column transforms into a scratch in 11 chunks of pixels and a sum over them; 96 x 160,
// 793 pixels, 75 us against 230 us.
#pragma once

#include "fft_generic.h"
#include "ssb_fused.h"

namespace stem {

constexpr int kGsEpt = 16;     // registers (complex) a thread holds of a pass
constexpr int kGsBatch = 64;   // pixels whose descriptors are gathered at once
constexpr int kGsRows = 4352;  // LDS elements of the rows: 34 KB, so that the registers (two waves per
                               // SIMD: at three, 36 registers spill), not LDS, set the residency

// threads of a workgroup: the last pass has at most one butterfly per thread
inline int gsum_threads(int ny) { return ny > 2048 ? 512 : 256; }

// The pixels of a batch with a pair in the column or its mirror: their packed sets, the offsets of
// their runs of the pruned array and the phase polynomials of both columns.
template <bool CHI0, bool PWRITE>
struct GsBatch {
  int4 set[kGsBatch];
  int32_t kd[kGsBatch];
  int64_t pd[PWRITE ? kGsBatch : 1], pm[PWRITE ? kGsBatch : 1];
  ChiRow cd[CHI0 ? 1 : kGsBatch], cm[CHI0 ? 1 : kGsBatch];
  int32_t n;
};

template <bool CHI0, bool PWRITE, int T>
__global__ void __launch_bounds__(T, 2) k_gsum(YArgs a, Optics o, GPlan p, int rb, int stride) {
  if (state_unready(a)) return;
  extern __shared__ __align__(16) float2 s_g[];  // twiddles, then rb rows
  __shared__ GsBatch<CHI0, PWRITE> sb;
  const int ny = p.n, nx = a.nx, nc = nx / 2 + 1;
  float2* tw = s_g;
  float2* buf = s_g + gen_tw_size(p);
  const int tid = threadIdx.x, lane = tid & 63;
  const int g = blockIdx.x % a.ngroups, c = blockIdx.x / a.ngroups;
  const bool mir = c > 0 && 2 * c < nx;
  const int kd_a = a.k0 + (int)((int64_t)(a.k1 - a.k0) * g / a.ngroups);
  const int kd_b = a.k0 + (int)((int64_t)(a.k1 - a.k0) * (g + 1) / a.ngroups);
  const uint64_t* mrow = a.cmask + (int64_t)(c / colset_width(ny)) * a.nmw;
  gen_twiddles(tw, (double2*)buf, p);
  const GPass& last = p.p[p.np - 1];
  float2 accd[kGsEpt], accm[kGsEpt];
#pragma unroll
  for (int q = 0; q < kGsEpt; ++q) accd[q] = accm[q] = make_float2(0.f, 0.f);
  unsigned cnt = 0, nld = 0;
  for (int w = kd_a >> 6; 64 * w < kd_b; ++w) {
    __syncthreads();  // the previous batch's descriptors are no longer read
    if (tid < 64) {
      const int kd = 64 * w + lane;
      bool on = kd >= kd_a && kd < kd_b && ((mrow[w] >> lane) & 1u);
      int4 raw = make_int4(0, 0, 0, 0);
      if (on) {
        raw = a.cst[(int64_t)kd * nc + c];
        ColSet d, m;
        unpack_colsets(raw, d, m);
        on = !d.empty() || !m.empty();  // a mask bit covers the columns of a whole set
      }
      const uint64_t bits = __ballot(on);
      if (on) {
        const int i = __builtin_popcountll(bits & ((1ull << lane) - 1));
        sb.set[i] = raw;
        sb.kd[i] = kd;
        if constexpr (PWRITE) {
          sb.pd[i] = a.poff[(int64_t)c * a.n_k + kd];
          sb.pm[i] = mir ? a.poff[(int64_t)(nx - c) * a.n_k + kd] : 0;
        }
        if constexpr (!CHI0) {
          const double2 k = a.kc[kd];
          const double kch = a.kchi[kd];
          const double qd = (double)signed_index(c, nx) * o.sx, qm = (double)signed_index(nx - c, nx) * o.sx;
          sb.cd[i] = chi_row(chi_column(o.lk * (k.x - qd), o), o.lk * k.y, -o.lk * o.sy, kch);
          sb.cm[i] = chi_row(chi_column(o.lk * (k.x - qm), o), o.lk * k.y, -o.lk * o.sy, kch);
        }
      }
      if (lane == 0) sb.n = __builtin_popcountll(bits);
    }
    __syncthreads();
    const int n = sb.n;
    float2 v[kGsEpt];
    // the first pass's inputs of the pixels i0 .. i0 + rb - 1 of the batch
    auto load = [&](int i0) {
      gen_radix(p.p[0].r, [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        gen_each<R, kGsEpt, T>(gen_tid(), p.p[0], rb, [&](int b, int row, int j) {
          if (i0 + row < n) {
            const float2* col = a.X + ((int64_t)(sb.kd[i0 + row] - a.xk0) * nc + c) * ny + j;
#pragma unroll
            for (int q = 0; q < R; ++q) v[b * R + q] = col[q * p.p[0].m];
            nld += R;
          } else {
#pragma unroll
            for (int q = 0; q < R; ++q) v[b * R + q] = make_float2(0.f, 0.f);
          }
        });
      });
    };
    if (n > 0) load(0);
    for (int i0 = 0; i0 < n; i0 += rb) {
      gen_radix(p.p[0].r, [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        const int t = gen_tid();
        gen_compute<R, kGsEpt, T, false>(t, v, tw, p.p[0], rb);
        gen_write<R, kGsEpt, T>(t, v, buf, stride, p.p[0], rb);
      });
      __syncthreads();
      if (i0 + rb < n) load(i0 + rb);
      for (int s = 1; s < p.np - 1; ++s) gen_pass<kGsEpt, T, true>(buf, stride, tw, p.p[s], rb);
      float2 u[kGsEpt];
      const int t = gen_tid(), lrow = gdiv(t, last.mm), lj = t - lrow * last.m;  // this thread's last butterfly
      gen_radix(last.r, [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        if (lrow < rb) {
          const float2* in = buf + lrow * stride;
          const float2* wt = tw + last.off + lj;  // ns = m: lj mod ns = lj
#pragma unroll
          for (int q = 0; q < R; ++q) u[q] = in[gpad(lj + q * last.m)];
#pragma unroll
          for (int q = 1; q < R; ++q) u[q] = cmul(u[q], wt[(q - 1) * last.ns]);
          gdft<R>(u);
        }
      });
      __syncthreads();  // the next pixels' first pass may overwrite the rows
      const int d = i0 + lrow;
      if (lrow < rb && d < n) {
        ColSet sd, sm;
        unpack_colsets(sb.set[d], sd, sm);
#pragma unroll
        for (int q = 0; q < kGsEpt; ++q) {
          if (q < last.r) {
            const int iy = signed_index(lj + q * last.m, ny);
            const int jy = 2 * iy == -ny ? iy : -iy;  // the mirrored frequency
            const bool hd = sd.has(iy), hm = sm.has(jy);
            cnt += (hd ? 1u : 0u) + (hm ? 1u : 0u);
            if constexpr (PWRITE) {
              if (hd) {
                const int64_t e = sb.pd[d] + set_rank(sd, iy);
                if (e >= 0 && e < a.pcap) a.pgw[e] = u[q];
              }
              if (hm) {
                const int64_t e = sb.pm[d] + set_rank(sm, jy);
                if (e >= 0 && e < a.pcap) a.pgw[e] = cconj(u[q]);
              }
            }
            if constexpr (CHI0) {
              // every phase factor is 1: a weight of 1 adds the value exactly, 0 adds nothing
              const float wd = hd ? 1.f : 0.f, wm = hm ? 1.f : 0.f;
              accd[q].x = fmaf(u[q].x, wd, accd[q].x);
              accd[q].y = fmaf(u[q].y, wd, accd[q].y);
              accm[q].x = fmaf(u[q].x, wm, accm[q].x);
              accm[q].y = fmaf(-u[q].y, wm, accm[q].y);
            } else {
              if (hd) {
                const float2 e = expi_rev(chi_row_eval(sb.cd[d], (double)iy));
                accd[q].x += u[q].x * e.x - u[q].y * e.y;
                accd[q].y += u[q].x * e.y + u[q].y * e.x;
              }
              if (hm) {
                const float2 e = expi_rev(chi_row_eval(sb.cm[d], (double)jy));
                accm[q].x += u[q].x * e.x + u[q].y * e.y;
                accm[q].y += u[q].x * e.y - u[q].y * e.x;
              }
            }
          }
        }
      }
    }
  }
  // the slots' sums added in order through the rows' LDS, then out: part[g], column-major [mx][my]
  float2* pgp = a.part + (int64_t)g * nx * ny;
  const int lrow = gdiv(tid, last.mm), lj = tid - lrow * last.m;
  for (int side = 0; side < (mir ? 2 : 1); ++side) {
    __syncthreads();
    if (lrow < rb) {
#pragma unroll
      for (int q = 0; q < kGsEpt; ++q)
        if (q < last.r) buf[lrow * stride + gpad(lj + q * last.m)] = side ? accm[q] : accd[q];
    }
    __syncthreads();
    for (int my = tid; my < ny; my += T) {
      float2 t = buf[gpad(my)];
      for (int r = 1; r < rb; ++r) t = cadd(t, buf[r * stride + gpad(my)]);
      float2* dst = side ? pgp + (int64_t)(nx - c) * ny + (my ? ny - my : 0) : pgp + (int64_t)c * ny + my;
      *dst = a.accumulate ? cadd(*dst, t) : t;
    }
  }
  unsigned long long cc = (unsigned long long)cnt + ((unsigned long long)nld << kLoadShift);
  for (int off = 32; off > 0; off >>= 1) cc += __shfl_xor(cc, off);
  const int64_t wid = (int64_t)blockIdx.x * (T / 64) + (tid >> 6);
  if (lane == 0) a.wcnt[wid] = a.accumulate ? a.wcnt[wid] + cc : cc;
}

// Pixel groups: about 2048 workgroups for a sum over all pixels at once (the GPU holds 512: enough
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

// pixels transformed together; 0 if ny has no plan
inline int gsum_rows(int ny, GPlan& p) {
  if (!gen_plan(ny, p)) return 0;
  const int T = gsum_threads(ny);
  int rb = gen_max_rows(p, T, kGsEpt);
  const int one = T / p.p[p.np - 1].m, lds = kGsRows / gen_stride(ny);
  rb = one < rb ? one : rb;
  rb = lds < rb ? lds : rb;
  return rb < kGsBatch ? rb : kGsBatch;
}

inline int launch_gsum(int ny, const YArgs& a, const Optics& o, int chi0, bool pwrite, hipStream_t s) {
  GPlan p;
  const int rb = gsum_rows(ny, p);
  if (rb < 1) return STEM_EINVAL;
  const int stride = gen_stride(ny);
  const size_t lds = gen_lds(p, rb, stride);
  const dim3 grid((unsigned)((a.nx / 2 + 1) * a.ngroups));
  STEM_TRACE("ssb_gsum", s);
  auto go = [&](auto c0, auto pw, auto t) {
    constexpr int T = decltype(t)::value;
    hipLaunchKernelGGL((k_gsum<decltype(c0)::value, decltype(pw)::value, T>), grid, dim3(T), lds, s, a, o, p, rb, stride);
  };
  auto by_threads = [&](auto c0, auto pw) {
    if (gsum_threads(ny) == 512) go(c0, pw, std::integral_constant<int, 512>{});
    else go(c0, pw, std::integral_constant<int, 256>{});
  };
  using T_ = std::true_type;
  using F_ = std::false_type;
  if (pwrite)
    chi0 ? by_threads(T_{}, T_{}) : by_threads(F_{}, T_{});
  else
    chi0 ? by_threads(T_{}, F_{}) : by_threads(F_{}, F_{});
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

}  // namespace stem

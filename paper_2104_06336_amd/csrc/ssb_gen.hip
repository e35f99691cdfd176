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
// Bound by vector arithmetic (VALU busy 0.85).  Measured (one MI355X, without aberrations): 1000 x 1000
// scan, 176 pixels, storing the values, 321 us against 1620 us for column transforms into a scratch in
// 11 chunks of pixels and a sum over them; 96 x 160, 793 pixels, 54 us against 230 us.  At two waves
// per SIMD (16 registers a pass for every plan), set tests of four comparisons and rows padded per 16
// elements it took 505 and 75 us.
#include "ssb_gen.h"

#include "trace.h"

namespace stem {

// Registers (complex) a thread holds of a pass: 12 for the plans of radices up to 12 (three waves per
// SIMD), else 16 (two).
static int gsum_ept(const GPlan& p) { return p.p[p.np - 1].r <= 12 ? 12 : 16; }
constexpr int kGsBatch = 64;   // pixels whose descriptors are gathered at once
constexpr int kGsRows = 4352;  // LDS elements of the rows where more than one fits: 34 KB, so that the
                               // registers, not LDS, set the residency (one padded row alone may be longer)

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

// A set for the tests and ranks of many frequencies iy = a0 + u: length of [a0, a1] (0 if empty), start and
// length of the hole in it.
struct RunSet {
  int a0;
  unsigned len, h0, hl;
  __device__ __forceinline__ explicit RunSet(const ColSet& s) {
    const int lo = max(s.a0, s.b0), hi = min(s.a1, s.b1);
    a0 = s.a0;
    len = s.a0 <= s.a1 ? (unsigned)(s.a1 - s.a0 + 1) : 0u;
    h0 = (unsigned)(lo - s.a0);
    hl = lo <= hi ? (unsigned)(hi - lo + 1) : 0u;
  }
  __device__ __forceinline__ bool has(int u) const { return (unsigned)u < len && (unsigned)u - h0 >= hl; }
  __device__ __forceinline__ unsigned size() const { return len - (len ? hl : 0u); }
  // position in the run of u in the set
  __device__ __forceinline__ unsigned rank(int u) const { return (unsigned)u - (hl && (unsigned)u >= h0 ? hl : 0u); }
};

template <bool CHI0, bool PWRITE, int T, int EPT>
__global__ void __launch_bounds__(T, EPT == 12 ? 3 : 2) k_gsum(YArgs a, Optics o, GPlan p, int rb, int stride) {
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
  const GPass p0 = p.p[0], last = p.p[p.np - 1];
  float2 accd[EPT], accm[EPT];
#pragma unroll
  for (int q = 0; q < EPT; ++q) accd[q] = accm[q] = make_float2(0.f, 0.f);
  unsigned cnt = 0, nld = 0;
  for (int w = kd_a >> 6; 64 * w < kd_b; ++w) {
    __syncthreads();  // the previous batch's descriptors are no longer read
    if (tid < 64) {
      const int kd = 64 * w + lane;
      bool on = kd >= kd_a && kd < kd_b && ((mrow[w] >> lane) & 1u);
      int4 raw = make_int4(0, 0, 0, 0);
      int64_t pd = 0, pm = 0;
      if (on) {
        raw = a.cst[(int64_t)kd * nc + c];
        ColSet d, m;
        unpack_colsets(raw, d, m);
        on = !d.empty() || !m.empty();  // a mask bit covers the columns of a whole set
        if constexpr (PWRITE) {
          pd = a.poff[(int64_t)c * a.n_k + kd];
          pm = mir ? a.poff[(int64_t)(nx - c) * a.n_k + kd] : 0;
          // runs outside the array are neither written nor summed (never with the layout's bound)
          on = on && pd >= 0 && pd + RunSet(d).size() <= a.pcap && pm >= 0 && pm + RunSet(m).size() <= a.pcap;
        }
      }
      const uint64_t bits = __ballot(on);
      if (on) {
        const int i = __builtin_popcountll(bits & ((1ull << lane) - 1));
        sb.set[i] = raw;
        sb.kd[i] = kd;
        if constexpr (PWRITE) {
          sb.pd[i] = pd;
          sb.pm[i] = pm;
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
    float2 v[EPT];
    // the first pass's inputs of the pixels i0 .. i0 + rb - 1 of the batch
    auto load = [&](int i0) {
      gen_radix<EPT>(p0.r, [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        gen_each<R, EPT, T>(gen_tid(), p0, rb, [&](int b, int row, int j) {
          if (i0 + row < n) {
            const float2* col = a.X + ((int64_t)(sb.kd[i0 + row] - a.xk0) * nc + c) * ny + j;
#pragma unroll
            for (int q = 0; q < R; ++q) v[b * R + q] = col[q * p0.m];
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
      gen_radix<EPT>(p0.r, [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        const int t = gen_tid();
        gen_compute<R, EPT, T, false>(t, v, tw, p0, rb);
        gen_write<R, EPT, T>(t, v, buf, stride, p0, rb);
      });
      __syncthreads();
      if (i0 + rb < n) load(i0 + rb);
      for (int s = 1; s < p.np - 1; ++s) {
        const GPass ps = p.p[s];
        gen_pass<EPT, T, true>(buf, stride, tw, ps, rb);
      }
      float2 u[EPT];
      const int t = gen_tid(), lrow = gdiv(t, last.mm), lj = t - lrow * last.m;  // this thread's last butterfly
      gen_radix<EPT>(last.r, [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        if (lrow < rb) {
          const float2* in = buf + lrow * stride + lj + gdiv(lj, last.mns) * last.rp;
          const float2* wt = tw + last.off + lj;  // ns = m: lj mod ns = lj
#pragma unroll
          for (int q = 0; q < R; ++q) u[q] = in[q * last.rq];
#pragma unroll
          for (int q = 1; q < R; ++q) u[q] = cmul(u[q], wt[(q - 1) * last.ns]);
          gdft<R>(u);
        }
      });
      __syncthreads();  // the next pixels' first pass may overwrite the rows
      const int d = i0 + lrow;
      if (lrow < rb && d < n) {
        ColSet cd, cm;
        unpack_colsets(sb.set[d], cd, cm);
        const RunSet sd(cd), sm(cm);
        float2 *wd_ = nullptr, *wm_ = nullptr;
        if constexpr (PWRITE) {
          wd_ = a.pgw + sb.pd[d];
          wm_ = a.pgw + sb.pm[d];
        }
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
          if (q < last.r) {
            const int my = lj + q * last.m;
            const int iy = 2 * my < ny ? my : my - ny;
            const int jy = 2 * my == ny ? iy : -iy;  // the mirrored frequency
            const int ud = iy - sd.a0, um = jy - sm.a0;
            const bool hd = sd.has(ud), hm = sm.has(um);
            cnt += (hd ? 1u : 0u) + (hm ? 1u : 0u);
            if constexpr (PWRITE) {
              if (hd) wd_[sd.rank(ud)] = u[q];
              if (hm) wm_[sm.rank(um)] = cconj(u[q]);
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
      for (int q = 0; q < EPT; ++q)
        if (q < last.r) buf[lrow * stride + lj + q * last.m] = side ? accm[q] : accd[q];
    }
    __syncthreads();
    for (int my = tid; my < ny; my += T) {
      float2 t = buf[my];
      for (int r = 1; r < rb; ++r) t = cadd(t, buf[r * stride + my]);
      float2* dst = side ? pgp + (int64_t)(nx - c) * ny + (my ? ny - my : 0) : pgp + (int64_t)c * ny + my;
      *dst = a.accumulate ? cadd(*dst, t) : t;
    }
  }
  unsigned long long cc = (unsigned long long)cnt + ((unsigned long long)nld << kLoadShift);
  for (int off = 32; off > 0; off >>= 1) cc += __shfl_xor(cc, off);
  const int64_t wid = (int64_t)blockIdx.x * (T / 64) + (tid >> 6);
  if (lane == 0) a.wcnt[wid] = a.accumulate ? a.wcnt[wid] + cc : cc;
}

int gsum_rows(int ny, GPlan& p) {
  if (!gen_plan(ny, p)) return 0;
  const int T = gsum_threads(ny);
  int rb = gen_max_rows(p, T, gsum_ept(p));
  const int one = T / p.p[p.np - 1].m, lds = kGsRows / p.len > 1 ? kGsRows / p.len : 1;
  rb = one < rb ? one : rb;
  rb = lds < rb ? lds : rb;
  return rb < kGsBatch ? rb : kGsBatch;
}

int launch_gsum(int ny, const YArgs& a, const Optics& o, int chi0, bool pwrite, hipStream_t s) {
  GPlan p;
  const int rb = gsum_rows(ny, p);
  if (rb < 1) return STEM_EINVAL;
  const int stride = p.len;
  const size_t lds = gen_lds(p, rb, stride);
  const dim3 grid((unsigned)((a.nx / 2 + 1) * a.ngroups));
  STEM_TRACE("ssb_gsum", s);
  auto go = [&](auto c0, auto pw, auto t, auto e) {
    constexpr int T = decltype(t)::value, EPT = decltype(e)::value;
    hipLaunchKernelGGL((k_gsum<decltype(c0)::value, decltype(pw)::value, T, EPT>), grid, dim3(T), lds, s, a, o, p, rb,
                       stride);
  };
  auto by_size = [&](auto c0, auto pw) {
    using I12 = std::integral_constant<int, 12>;
    using I16 = std::integral_constant<int, 16>;
    using I256 = std::integral_constant<int, 256>;
    using I512 = std::integral_constant<int, 512>;
    if (gsum_threads(ny) == 512) gsum_ept(p) == 12 ? go(c0, pw, I512{}, I12{}) : go(c0, pw, I512{}, I16{});
    else gsum_ept(p) == 12 ? go(c0, pw, I256{}, I12{}) : go(c0, pw, I256{}, I16{});
  };
  using T_ = std::true_type;
  using F_ = std::false_type;
  if (pwrite)
    chi0 ? by_size(T_{}, T_{}) : by_size(F_{}, T_{});
  else
    chi0 ? by_size(T_{}, F_{}) : by_size(F_{}, F_{});
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

}  // namespace stem

// The transforms of a fit (SSBPhase and its adjoint) at the scan lengths the wavefront FFT does not
// take: radix 4, 2, 3, 5 passes, one real row per transform.
//
// dL/dc leaves in FP64 but carries the rounding of these FP32 transforms.  Those of fft_generic.h round
// differently (two real rows share a complex transform, radices up to 16) and move dL/dc by 0.6e-7 to
// 4e-7 of its value (12 geometries, as far as either is from the gradient in FP64); a fit keeps these in
// its forward and its adjoint, so that its gradients stay what they were bit for bit, at the cost of their
// speed (144 x 40, 707 pixels: a gradient takes 770 us against 290 us).
//
// A workgroup transforms RB = max(1, 4096/N) rows at once in LDS with a Stockham autosort FFT; every thread
// reads all its butterflies' inputs before the workgroup barrier and writes after it, so one LDS buffer
// serves each pass in place.  Twiddles come from an LDS table of W_N^t, t < N, evaluated in FP64 with the
// angle 2t/N and rounded to FP32; the exponent q (j mod Ns) N/(Ns R) is an integer below N.
#include "common.h"
#include "fft_generic.h"
#include "kernels.h"
#include "trace.h"

namespace stem {

namespace fit {

constexpr int kMaxPasses = 12;

struct GPlan {
  int32_t n;
  int32_t np;
  int32_t r[kMaxPasses];
};

// N = 2^a 3^b 5^c with 2 <= N <= kGenMax, factored into passes; false otherwise.
static bool gen_plan(int n, GPlan& p) {
  if (n < 2 || n > kGenMax) return false;
  p.n = n;
  p.np = 0;
  int m = n;
  while (m % 4 == 0 && p.np < kMaxPasses) { p.r[p.np++] = 4; m /= 4; }
  while (m % 2 == 0 && p.np < kMaxPasses) { p.r[p.np++] = 2; m /= 2; }
  while (m % 3 == 0 && p.np < kMaxPasses) { p.r[p.np++] = 3; m /= 3; }
  while (m % 5 == 0 && p.np < kMaxPasses) { p.r[p.np++] = 5; m /= 5; }
  return m == 1;
}

__host__ __device__ static inline int gen_rows_per_block(int n) { return n >= kGenMax ? 1 : kGenMax / n; }

// tw[t] = exp(-2 pi i t / n), t < n (FP64 evaluation, FP32 rounding); every thread of the workgroup
// takes part
__device__ __forceinline__ void gen_twiddles(float2* tw, int n) {
  for (int t = threadIdx.x; t < n; t += blockDim.x) {
    double s, c;
    sincospi(2.0 * (double)t / (double)n, &s, &c);
    tw[t] = make_float2((float)c, (float)-s);
  }
}

// length-R DFTs in registers (forward sign), natural order in and out
__device__ __forceinline__ void gdft2(float2* v) {
  const float2 a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}

__device__ __forceinline__ void gdft4(float2* v) {
  const float2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]), t2 = cadd(v[1], v[3]), t3 = csub(v[1], v[3]);
  v[0] = cadd(t0, t2);
  v[2] = csub(t0, t2);
  v[1] = cadd(t1, cmul_mi(t3));
  v[3] = csub(t1, cmul_mi(t3));
}

// One Stockham pass of radix R over rb rows of length n at buf[row * n + i] (blockDim.x ==
// kGenThreads).  The twiddle exponent q (j mod Ns) n/(Ns R) is below n.
template <int R>
__device__ __forceinline__ void gen_pass(float2* buf, const float2* tw, int n, int rb, int ns) {
  const int m = n / R;               // butterflies per row
  const int tstride = n / (ns * R);  // twiddle index step of exponent 1
  const int total = rb * m;
  // butterflies per thread: rb n <= kGenMax elements make at most kGenMax / R butterflies
  constexpr int kMaxB = (kGenMax / R + kGenThreads - 1) / kGenThreads;
  float2 v[kMaxB][R];
#pragma unroll
  for (int b = 0; b < kMaxB; ++b) {
    const int g = threadIdx.x + b * kGenThreads;
    if (g < total) {
      const int row = g / m, j = g % m;
      const float2* in = buf + row * n;
      const int k = j % ns;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        float2 x = in[j + q * m];
        if (q > 0 && ns > 1) x = cmul(x, tw[q * k * tstride]);
        v[b][q] = x;
      }
      if constexpr (R == 2) gdft2(v[b]);
      else if constexpr (R == 3) gdft3(v[b]);
      else if constexpr (R == 4) gdft4(v[b]);
      else gdft5(v[b]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < kMaxB; ++b) {
    const int g = threadIdx.x + b * kGenThreads;
    if (g < total) {
      const int row = g / m, j = g % m;
      float2* out = buf + row * n;
      const int base = (j / ns) * ns * R + (j % ns);
#pragma unroll
      for (int q = 0; q < R; ++q) out[base + q * ns] = v[b][q];
    }
  }
  __syncthreads();
}

// Forward FFT of rb rows of length p.n in buf (LDS), in place; tw from gen_twiddles.
__device__ __forceinline__ void gen_fft(float2* buf, const float2* tw, const GPlan& p, int rb) {
  int ns = 1;
  for (int s = 0; s < p.np; ++s) {
    const int r = p.r[s];
    if (r == 4) gen_pass<4>(buf, tw, p.n, rb, ns);
    else if (r == 2) gen_pass<2>(buf, tw, p.n, rb, ns);
    else if (r == 3) gen_pass<3>(buf, tw, p.n, rb, ns);
    else gen_pass<5>(buf, tw, p.n, rb, ns);
    ns *= r;
  }
}


__global__ void __launch_bounds__(kGenThreads) k_fit_fft(RowFftArgs a, GPlan p, int inv, int in_mode, int out_mode) {
  extern __shared__ float2 s_g[];  // twiddles [n], then rb rows of n
  const int n = p.n, rb = gen_rows_per_block(n);
  float2* tw = s_g;
  float2* buf = s_g + n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (in_mode == IN_C64_SUM && a.stats && blockIdx.x == 0) {
    // the fused sums' per-wave counters: pair count below bit 40, 8-byte loads above
    __shared__ unsigned long long s_red[2][kGenThreads / 64];
    unsigned long long c = 0, l = 0;
    for (int64_t i = threadIdx.x; i < a.nwcnt; i += blockDim.x) {
      c += a.wcnt[i] & ((1ull << 40) - 1);
      l += a.wcnt[i] >> 40;
    }
    for (int off = 32; off > 0; off >>= 1) {
      c += __shfl_xor(c, off);
      l += __shfl_xor(l, off);
    }
    if (lane == 0) {
      s_red[0][wave] = c;
      s_red[1][wave] = l;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
      unsigned long long t = 0, u = 0;
      for (int w = 0; w < kGenThreads / 64; ++w) {
        t += s_red[0][w];
        u += s_red[1][w];
      }
      a.stats[threadIdx.x] = threadIdx.x == 0   ? t
                             : threadIdx.x == 1 ? (a.part_seg ? (unsigned long long)a.part_seg[a.nrows]
                                                              : (unsigned long long)a.stats_groups)
                             : threadIdx.x == 2 ? 8ull * u
                                                : (unsigned long long)a.stats_chunks;
    }
    if (threadIdx.x == 4 && a.ready_out) *a.ready_out = a.ready_val;
  }
  gen_twiddles(tw, n);
  __syncthreads();
  const int64_t nbatch = (a.nrows + rb - 1) / rb;
  const bool transposed = out_mode == OUT_T_C64 || out_mode == OUT_X;
  const int nh = n / 2 + 1;
  for (int64_t bt = blockIdx.x; bt < nbatch; bt += gridDim.x) {
    const int64_t r0 = bt * rb;
    for (int e = threadIdx.x; e < rb * n; e += blockDim.x) {
      const int rl = e / n, i = e % n;
      const int64_t r = r0 + rl;
      float2 x = make_float2(0.f, 0.f);
      if (r < a.nrows) {
        const int64_t el = r * n + i;
        if (in_mode == IN_C64) {
          x = a.in_c[el];
        } else if (in_mode == IN_C64_SUM) {
          if (a.part_seg) {
            const int64_t q0 = min(max(a.part_seg[r], (int64_t)0), a.part_seg_rows);
            const int64_t q1 = min(max(a.part_seg[r + 1], q0), a.part_seg_rows);
            for (int64_t q = q0; q < q1; ++q) x = cadd(x, a.in_c[q * n + i]);
          } else {
            for (int q = 0; q < a.nparts; ++q) x = cadd(x, a.in_c[(int64_t)q * a.part_stride + el]);
          }
          if (a.norm_cnt) {
            const int32_t cnt = a.norm_cnt[el];
            x = cnt > 0 ? make_float2(x.x / (float)cnt, x.y / (float)cnt) : make_float2(0.f, 0.f);
          }
          if (a.sum_out) a.sum_out[el] = x;
        } else if (in_mode == IN_F32_PAIR) {
          x.x = a.in_f0[el] * a.s0;
          x.y = a.in_f1 ? a.in_f1[el] * a.s1 : 0.f;
        } else if (in_mode == IN_U8) {
          x.x = (float)((const uint8_t*)a.in_u)[el];
        } else {
          x.x = (float)((const uint16_t*)a.in_u)[el];
        }
      }
      buf[e] = inv ? cconj(x) : x;
    }
    __syncthreads();
    gen_fft(buf, tw, p, rb);
    for (int e = threadIdx.x; e < rb * n; e += blockDim.x) {
      // transposed outputs rows-fastest, the others along the row
      const int rl = transposed ? e % rb : e / n, m = transposed ? e / rb : e % n;
      const int64_t r = r0 + rl;
      if (r >= a.nrows) continue;
      const float2 y = buf[rl * n + m];
      const float2 v = cmul(inv ? cconj(y) : y, a.osc);
      // (the same as a chain of conditions compiles to a slower kernel: 720 x 360, 176 pixels, a fit's forward 1117
      // instead of 1068 us)
      switch (out_mode) {
        case OUT_ROW_C64: a.out_c[r * n + m] = v; break;
        case OUT_ROW_IM: a.out_f[r * n + m] = v.y; break;
        case OUT_T_C64: a.out_c[(int64_t)m * a.out_stride + r] = v; break;
        default:  // OUT_X
          if (m < nh) {
            const int64_t kd = r / a.xrows, y_ = r % a.xrows;
            a.out_c[(kd * nh + m) * a.xrows + y_] = v;
          }
      }
    }
    __syncthreads();
  }
}

}  // namespace fit

int launch_fit_row_fft(int n, bool inverse, RowIn in, RowOut out, const RowFftArgs& a, hipStream_t stream) {
  if (a.nrows <= 0) return STEM_OK;
  // the modes a fit uses
  if (in == IN_F64_PAIR || in == IN_HALF_C64 || out == OUT_ROW_RE) return STEM_EINVAL;
  if (fast_length(n) && in != IN_U8 && in != IN_U16 && out != OUT_X)
    return launch_row_fft(n, inverse, in, out, a, stream);
  STEM_TRACE(a.tag ? a.tag : "row_fft", stream);
  fit::GPlan p;
  if (!fit::gen_plan(n, p)) return STEM_EINVAL;
  const int rb = fit::gen_rows_per_block(n);
  const int64_t batches = (a.nrows + rb - 1) / rb;
  const size_t lds = (size_t)(n + rb * n) * sizeof(float2);
  const int res = resident_blocks((const void*)fit::k_fit_fft, kGenThreads, lds);
  const int64_t cap = res > 0 ? res : 1024;
  hipLaunchKernelGGL(fit::k_fit_fft, dim3((unsigned)(batches < cap ? batches : cap)), dim3(kGenThreads), lds, stream, a,
                     p, inverse ? 1 : 0, (int)in, (int)out);
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

}  // namespace stem

// Batched row FFTs (power-of-two lengths 32..1024) and the centre-of-mass DPC path
// (Eq. 4 and the regularised Fourier gradient descent of Sec. V).
//
// k_row_fft: a workgroup of W = 8 waves (4 when there are too few rows to give every CU a
// workgroup); each wave transforms B = 1024/N rows at a time with the wavefront FFT of
// fft_wave.h.  Row-major outputs are stored straight from registers; transposed outputs
// (element (r, m) -> out[m*stride + r]) are first staged in the waves' LDS buffers so that the
// workgroup writes runs of W B consecutive rows per frequency.
#include <memory>
#include <mutex>
#include <new>
#include <type_traits>

#include "common.h"
#include "fft_generic.h"
#include "fft_wave.h"
#include "geom.h"
#include "kernels.h"
#include "trace.h"

namespace stem {

constexpr int kWaveStride = kFftLds + 4;  // float2 per wave buffer; the +4 staggers LDS banks

// SUM: the input is the sum of a.nparts partial planes (in_mode IN_C64_SUM), read four at a time;
// a separate instantiation, so that the other input modes keep their lower register count.  SEG
// (with SUM): the partials are segments, row r adding rows a.part_seg[r] .. a.part_seg[r+1]-1.
template <int N, bool INV, int W, bool SUM, bool SEG = false>
__global__ void __launch_bounds__(64 * W) k_row_fft(RowFftArgs a, int in_mode, int out_mode) {
  constexpr int kRowThreads = 64 * W;
  __shared__ float2 s_tw[1024];
  __shared__ float2 s_buf[W * kWaveStride];
  constexpr int B = 1024 / N;
  constexpr int TR = W * B;  // rows per tile
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if constexpr (SUM) {
    if (a.stats && blockIdx.x == 0) {
      // every thread of the first workgroup sums a strided share, four loads in flight
      // per wave: pair count below bit 40, 8-byte loads above
      __shared__ unsigned long long s_red[2][W];
      constexpr unsigned long long kLow = (1ull << 40) - 1;
      unsigned long long c0 = 0, c1 = 0, l0 = 0, l1 = 0;
      for (int64_t i = threadIdx.x; i < a.nwcnt; i += 2 * kRowThreads) {
        const unsigned long long u = a.wcnt[i];
        c0 += u & kLow;
        l0 += u >> 40;
        if (i + kRowThreads < a.nwcnt) {
          const unsigned long long v = a.wcnt[i + kRowThreads];
          c1 += v & kLow;
          l1 += v >> 40;
        }
      }
      unsigned long long c = c0 + c1, l = l0 + l1;
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
        for (int w = 0; w < W; ++w) {
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
  }
  fill_twiddles(s_tw, threadIdx.x, kRowThreads);
  __syncthreads();
  float2* buf = s_buf + wave * kWaveStride;
  const int64_t ntiles = (a.nrows + TR - 1) / TR;
  const bool transposed = out_mode == OUT_T_C64;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t r0 = tile * TR + wave * B;
    float2 v[16];
    if constexpr (SUM) {
      // partial sums added in a fixed order; the 64 loads of four partials are issued together
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = make_float2(0.f, 0.f);
      auto load_part = [&](int p, float2* t) {
        const float2* src = a.in_c + (int64_t)p * a.part_stride;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          int b, n;
          fft_in_index<N>(lane, i, b, n);
          const int64_t r = r0 + b;
          t[i] = r < a.nrows ? src[r * N + n] : make_float2(0.f, 0.f);
        }
      };
      if constexpr (SEG) {
        // segments: row r adds rows part_seg[r] .. part_seg[r + 1] - 1, in order (a lane's 16
        // elements are of one row); the wave runs to the largest count among its rows
        int b, n;
        fft_in_index<N>(lane, 0, b, n);
        const int64_t r = r0 + b;
        const int64_t s0 = r < a.nrows ? min(max(a.part_seg[r], (int64_t)0), a.part_seg_rows) : 0;
        const int sn = r < a.nrows ? (int)(min(max(a.part_seg[r + 1], s0), a.part_seg_rows) - s0) : 0;
        int most = sn;
        for (int off = 32; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off));
        for (int q = 0; q < most; ++q) {
          float2 t[16];
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            fft_in_index<N>(lane, i, b, n);
            t[i] = q < sn ? a.in_c[(int64_t)(s0 + q) * N + n] : make_float2(0.f, 0.f);
          }
#pragma unroll
          for (int i = 0; i < 16; ++i) v[i] = cadd(v[i], t[i]);
        }
      } else {
        int p = 0;
        for (; p + 4 <= a.nparts; p += 4) {
          float2 t[4][16];
#pragma unroll
          for (int k = 0; k < 4; ++k) load_part(p + k, t[k]);
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = cadd(v[i], t[k][i]);
        }
        for (; p < a.nparts; ++p) {
          float2 t[16];
          load_part(p, t);
#pragma unroll
          for (int i = 0; i < 16; ++i) v[i] = cadd(v[i], t[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        int b, n;
        fft_in_index<N>(lane, i, b, n);
        const int64_t r = r0 + b;
        if (a.norm_cnt && r < a.nrows) {
          const int32_t c = a.norm_cnt[r * N + n];
          v[i] = c > 0 ? make_float2(v[i].x / (float)c, v[i].y / (float)c) : make_float2(0.f, 0.f);
        }
        if (a.sum_out && r < a.nrows) a.sum_out[r * N + n] = v[i];
        if (INV) v[i] = cconj(v[i]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        int b, n;
        fft_in_index<N>(lane, i, b, n);
        const int64_t r = r0 + b;
        float2 x = make_float2(0.f, 0.f);
        if (r < a.nrows) {
          const int64_t e = r * N + n;
          if (in_mode == IN_C64) {
            x = a.in_c[e];
          } else if (in_mode == IN_HALF_C64) {
            // Hermitian row from its first N/2 + 1 entries: x(N - m) = conj x(m)
            const float2* hr = a.in_c + r * (N / 2 + 1);
            x = 2 * n <= N ? hr[n] : cconj(hr[N - n]);
          } else if (in_mode == IN_F32_PAIR) {
            x.x = a.in_f0[e] * a.s0;
            x.y = a.in_f1 ? a.in_f1[e] * a.s1 : 0.f;
          } else {
            x.x = (float)(a.in_d0[e] * (double)a.s0);
            x.y = a.in_d1 ? (float)(a.in_d1[e] * (double)a.s1) : 0.f;
          }
        }
        v[i] = INV ? cconj(x) : x;
      }
    }
    wave_fft<N>(v, buf, s_tw, lane);
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = cmul(INV ? cconj(v[i]) : v[i], a.osc);
    if (!transposed) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        int b, m;
        fft_out_index<N>(lane, i, b, m);
        const int64_t r = r0 + b;
        if (r < a.nrows) {
          const int64_t e = r * N + m;
          if (out_mode == OUT_ROW_C64) a.out_c[e] = v[i];
          else if (out_mode == OUT_ROW_RE) a.out_f[e] = v[i].x;
          else a.out_f[e] = v[i].y;
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        int b, m;
        fft_out_index<N>(lane, i, b, m);
        buf[fft_pad(b * N + m)] = v[i];
      }
      __syncthreads();
      for (int u = threadIdx.x; u < TR * N; u += kRowThreads) {
        const int m = u / TR, rl = u % TR;
        const int w = rl / B, b = rl % B;
        const int64_t r = tile * TR + rl;
        if (r < a.nrows) {
          a.out_c[(int64_t)m * a.out_stride + r] = s_buf[w * kWaveStride + fft_pad(b * N + m)];
        }
      }
      __syncthreads();
    }
  }
}

template <int N, int W>
static void launch_nw(bool inv, const RowFftArgs& a, int in, int out, hipStream_t s) {
  const int64_t tr = W * (1024 / N);
  const int64_t tiles = (a.nrows + tr - 1) / tr;
  const dim3 grid((unsigned)(tiles < 2048 ? tiles : 2048));
  if (in == IN_C64_SUM && a.part_seg) {
    if (inv)
      hipLaunchKernelGGL((k_row_fft<N, true, W, true, true>), grid, dim3(64 * W), 0, s, a, in, out);
    else
      hipLaunchKernelGGL((k_row_fft<N, false, W, true, true>), grid, dim3(64 * W), 0, s, a, in, out);
  } else if (in == IN_C64_SUM) {
    if (inv)
      hipLaunchKernelGGL((k_row_fft<N, true, W, true>), grid, dim3(64 * W), 0, s, a, in, out);
    else
      hipLaunchKernelGGL((k_row_fft<N, false, W, true>), grid, dim3(64 * W), 0, s, a, in, out);
  } else if (inv) {
    hipLaunchKernelGGL((k_row_fft<N, true, W, false>), grid, dim3(64 * W), 0, s, a, in, out);
  } else {
    hipLaunchKernelGGL((k_row_fft<N, false, W, false>), grid, dim3(64 * W), 0, s, a, in, out);
  }
}

template <int N>
static void launch_n(bool inv, const RowFftArgs& a, int in, int out, hipStream_t s) {
  // fewer than two 8-wave tiles per CU: 4-wave workgroups spread the rows over more CUs
  if (a.nrows < 2 * 256 * 8 * (1024 / N))
    launch_nw<N, 4>(inv, a, in, out, s);
  else
    launch_nw<N, 8>(inv, a, in, out, s);
}

// ---------------------------------------------------------------------------------------------
// Batched row FFTs of the lengths the wavefront FFT does not take (fft_generic.h): a workgroup
// loads RB rows into LDS (the input modes of k_row_fft), transforms them and writes them (its output
// modes), grid-stride over batches of rows, its twiddles filled once.  Transposed outputs are written
// rows-fastest (runs of RB consecutive rows per frequency).  RB is what LDS holds of 4096 elements,
// less where that would leave compute units without a workgroup (1000 rows of 1000: 3 rows each; one row
// each takes 16 against 19 us, but 35 against 33 us where partials are summed).

constexpr int kGenRadices[11] = {2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16};

// The radices of n, ascending, as few as possible (at least two) and then with the smallest sum.
static void gen_factor(int n, int from, int depth, int* cur, int* best, int& best_np, int& best_sum) {
  if (n == 1) {
    int sum = 0;
    for (int i = 0; i < depth; ++i) sum += cur[i];
    if (depth >= 2 && (depth < best_np || (depth == best_np && sum < best_sum))) {
      best_np = depth;
      best_sum = sum;
      for (int i = 0; i < depth; ++i) best[i] = cur[i];
    }
    return;
  }
  if (depth >= kGenMaxPasses || depth >= best_np) return;
  for (int i = from; i < 11 && kGenRadices[i] <= n; ++i) {
    if (n % kGenRadices[i]) continue;
    cur[depth] = kGenRadices[i];
    gen_factor(n / kGenRadices[i], i, depth + 1, cur, best, best_np, best_sum);
  }
}

// Lanes of a group of g that share a bank of 8 bytes (g banks), worst bank, for element positions pos.
template <typename F>
static int bank_depth(int g, F&& pos) {
  int n[32] = {}, most = 0;
  for (int l = 0; l < g; ++l) {
    const int k = ++n[pos(l) % g];
    most = k > most ? k : most;
  }
  return most;
}

// The padding per block of ns r elements of the layout between a pass (ns, r) and the next: the one of
// at most an eighth of the block (at least 1) whose writes and reads share banks least, over the first 16
// and 32 lanes.
static int gen_pad(int ns, int r) {
  const int blk = ns * r, lim = blk / 8 > 1 ? (blk / 8 < 32 ? blk / 8 : 31) : 1;
  int best = 0, cost = 1 << 30;
  for (int w = 0; w <= lim; ++w) {
    int c = 0;
    for (int g = 16; g <= 32; g += 16) {
      c += bank_depth(g, [&](int l) { return l + l / ns * (ns * (r - 1) + w); });
      c += bank_depth(g, [&](int l) { return l + l / blk * w; });
    }
    if (c < cost) {
      cost = c;
      best = w;
    }
  }
  return best;
}

static bool gen_make_plan(int n, GPlan& p) {
  int cur[kGenMaxPasses], best[kGenMaxPasses], np = kGenMaxPasses + 1, sum = 0;
  gen_factor(n, 0, 0, cur, best, np, sum);
  if (np > kGenMaxPasses) return false;
  p.n = n;
  p.np = np;
  p.ntw = n - best[0];
  p.len = n;
  p.mn = gmagic(n);
  int ns = 1, rp = 0;
  for (int s = 0; s < np; ++s) {
    GPass& q = p.p[s];
    q.r = best[s];
    q.m = n / q.r;
    q.ns = ns;
    q.off = s ? ns - best[0] : 0;  // passes 1 .. s-1 hold ns (r - 1) entries each
    q.step = n / (ns * q.r);
    q.rp = rp;
    q.rq = q.m + q.m / ns * rp;
    q.wp = s < np - 1 ? gen_pad(ns, q.r) : 0;
    q.mm = gmagic(q.m);
    q.mns = gmagic(q.ns);
    ns *= q.r;
    rp = q.wp;
    p.len = n + n / ns * rp > p.len ? n + n / ns * rp : p.len;
  }
  return true;
}

bool gen_plan(int n, GPlan& p) {
  if (n < 4 || n > kGenMax) return false;
  static std::mutex mu;
  static std::unique_ptr<GPlan> plans[kGenMax + 1];
  {
    int m = n;
    while (m % 2 == 0) m /= 2;
    while (m % 3 == 0) m /= 3;
    while (m % 5 == 0) m /= 5;
    if (m != 1) return false;
  }
  std::lock_guard<std::mutex> lk(mu);
  if (!plans[n]) {
    GPlan q;
    if (!gen_make_plan(n, q)) return false;
    plans[n].reset(new (std::nothrow) GPlan(q));
    if (!plans[n]) {
      p = q;
      return true;
    }
  }
  p = *plans[n];
  return true;
}

bool scan_length_ok(int n) {
  if (fast_length(n)) return true;
  GPlan p;
  return n >= 16 && n % 2 == 0 && gen_plan(n, p);
}

constexpr int kGenEpt = 30;  // registers (complex) of a thread of the row passes: 4096 elements in any plan

// SEG: IN_C64_SUM over segments (a.part_seg)
template <int IN, bool SEG>
__global__ void __launch_bounds__(kGenThreads) k_grow_fft(RowFftArgs a, GPlan p, int rb, int inv, int out_mode) {
  extern __shared__ __align__(16) float2 s_g[];  // twiddles, then rb rows
  const int n = p.n, stride = p.len;
  float2* tw = s_g;
  float2* buf = s_g + gen_tw_size(p);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (IN == IN_C64_SUM && a.stats && blockIdx.x == 0) {
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
  gen_twiddles(tw, (double2*)buf, p);
  const int64_t nbatch = (a.nrows + rb - 1) / rb;
  const bool transposed = out_mode == OUT_T_C64;
  const uint32_t mrb = rb == 1 ? 0u : (uint32_t)((0x100000000ull + rb - 1) / rb);
  for (int64_t bt = blockIdx.x; bt < nbatch; bt += gridDim.x) {
    const int64_t r0 = bt * rb;
    // eight elements' loads in flight per thread (past the last element or row an in-range one is
    // loaded again)
    constexpr int U = 8;
    for (int e0 = threadIdx.x; e0 < rb * n; e0 += U * kGenThreads) {
      int64_t el[U];
      int pos[U];
      float2 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = min(e0 + u * kGenThreads, rb * n - 1);
        const int rl = gdiv(e, p.mn), i = e - rl * n;
        el[u] = min(r0 + rl, a.nrows - 1) * n + i;
        pos[u] = rl * stride + i;
      }
      if constexpr (IN == IN_C64) {
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = a.in_c[el[u]];
      } else if constexpr (IN == IN_F32_PAIR) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          x[u] = make_float2(a.in_f0[el[u]] * a.s0, a.in_f1 ? a.in_f1[el[u]] * a.s1 : 0.f);
      } else if constexpr (IN == IN_F64_PAIR) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          x[u] = make_float2((float)(a.in_d0[el[u]] * (double)a.s0),
                             a.in_d1 ? (float)(a.in_d1[el[u]] * (double)a.s1) : 0.f);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = make_float2(0.f, 0.f);
        if constexpr (SEG) {
          int64_t q0[U];
          int qn[U], most = 0;
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int64_t r = min(r0 + gdiv(min(e0 + u * kGenThreads, rb * n - 1), p.mn), a.nrows - 1);
            const int64_t s0 = min(max(a.part_seg[r], (int64_t)0), a.part_seg_rows);
            qn[u] = (int)(min(max(a.part_seg[r + 1], s0), a.part_seg_rows) - s0);
            q0[u] = s0 * n + (el[u] - r * n);
            most = max(most, qn[u]);
          }
          for (int q = 0; q < most; ++q)
#pragma unroll
            for (int u = 0; u < U; ++u)
              if (q < qn[u]) x[u] = cadd(x[u], a.in_c[q0[u] + (int64_t)q * n]);
        } else {
          // four partials' loads together, added in order
          for (int q = 0; q < a.nparts; q += 4) {
            float2 t[4][U];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const float2* src = a.in_c + min(q + k, a.nparts - 1) * a.part_stride;
#pragma unroll
              for (int u = 0; u < U; ++u) t[k][u] = src[el[u]];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
              for (int u = 0; u < U; ++u)
                if (q + k < a.nparts) x[u] = cadd(x[u], t[k][u]);
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (a.norm_cnt) {
            const int32_t cnt = a.norm_cnt[el[u]];
            x[u] = cnt > 0 ? make_float2(x[u].x / (float)cnt, x[u].y / (float)cnt) : make_float2(0.f, 0.f);
          }
          if (a.sum_out) a.sum_out[el[u]] = x[u];  // an element loaded again is stored again, the same
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) buf[pos[u]] = inv ? cconj(x[u]) : x[u];
    }
    __syncthreads();
    gen_pass<kGenEpt, kGenThreads, false>(buf, stride, tw, p.p[0], rb);
    for (int s = 1; s < p.np; ++s) {
      const GPass ps = p.p[s];
      gen_pass<kGenEpt, kGenThreads, true>(buf, stride, tw, ps, rb);
    }
    for (int e = threadIdx.x; e < rb * n; e += kGenThreads) {
      // transposed outputs rows-fastest, the others along the row
      const int hi = transposed ? gdiv(e, mrb) : gdiv(e, p.mn);
      const int rl = transposed ? e - hi * rb : hi, m = transposed ? hi : e - hi * n;
      const int64_t r = r0 + rl;
      if (r >= a.nrows) continue;
      const float2 y = buf[rl * stride + m];
      const float2 v = cmul(inv ? cconj(y) : y, a.osc);
      if (out_mode == OUT_ROW_C64) a.out_c[r * n + m] = v;
      else if (out_mode == OUT_ROW_RE) a.out_f[r * n + m] = v.x;
      else if (out_mode == OUT_ROW_IM) a.out_f[r * n + m] = v.y;
      else a.out_c[(int64_t)m * a.out_stride + r] = v;
    }
    __syncthreads();
  }
}

int gen_fft_rows(const GPlan& p, int64_t nrows) {
  const int most = gen_max_rows(p, kGenThreads, kGenEpt);
  const int64_t fill = nrows / 256 > 1 ? nrows / 256 : 1;
  int64_t rb = kGenMax / p.n;
  rb = rb > most ? most : rb;
  return (int)(rb > fill ? fill : rb);
}

static int launch_generic(int n, bool inverse, RowIn in, RowOut out, const RowFftArgs& a, hipStream_t stream) {
  GPlan p;
  if (!gen_plan(n, p)) return STEM_EINVAL;
  const int rb = gen_fft_rows(p, a.nrows);
  if (rb < 1) return STEM_EINVAL;
  const int64_t batches = (a.nrows + rb - 1) / rb;
  const size_t lds = gen_lds(p, rb, p.len);
  auto go = [&](auto mode, auto seg) {
    const auto fn = k_grow_fft<decltype(mode)::value, decltype(seg)::value>;
    const int res = resident_blocks((const void*)fn, kGenThreads, lds);
    const int64_t cap = res > 0 ? res : 1024;
    hipLaunchKernelGGL(fn, dim3((unsigned)(batches < cap ? batches : cap)), dim3(kGenThreads), lds, stream, a, p,
                       rb, inverse ? 1 : 0, (int)out);
  };
  using T_ = std::true_type;
  using F_ = std::false_type;
  if (in == IN_C64) go(std::integral_constant<int, IN_C64>{}, F_{});
  else if (in == IN_F32_PAIR) go(std::integral_constant<int, IN_F32_PAIR>{}, F_{});
  else if (in == IN_F64_PAIR) go(std::integral_constant<int, IN_F64_PAIR>{}, F_{});
  else if (in != IN_C64_SUM) return STEM_EINVAL;
  else if (a.part_seg) go(std::integral_constant<int, IN_C64_SUM>{}, T_{});
  else go(std::integral_constant<int, IN_C64_SUM>{}, F_{});
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

// ---------------------------------------------------------------------------------------------
// Row transform of the binned counts at any length: real rows r = kd ny + y of n counts, X[kd][m][y] for
// m <= n/2.  Two real rows make one complex transform; the workgroup splits the 2 RB half spectra from
// LDS and writes them in runs of 2 RB consecutive y (16-byte pairs: ny is even, so a pair is of one
// pixel).  The first pass reads the counts straight from global memory (neighbouring threads,
// neighbouring counts).  Workgroups of 512 threads with up to 64 KB of rows, two per compute unit;
// RB is a power of two, so that a thread keeps its row pair through the write loop.
//
// Bound by vector arithmetic and latency (VALU busy 0.64).  Measured (one MI355X): 1000 x 1000 scan, 176
// pixels of 8-bit counts, 299 us against 1640 us for one real row per complex transform written in runs of
// four; 96 x 160, 793 pixels of 16-bit counts, 26 us against 159 us.  Without the next tile's counts in
// flight and with rows padded per 16 elements (three operations per LDS address, twice the bank
// conflicts) the first took 473 us.
constexpr int kGenXThreads = 512;
constexpr int kGenXEpt = 20;

template <typename DT>
__global__ void __launch_bounds__(kGenXThreads, 4) k_grow_x(const DT* __restrict__ D, GPlan p, int lrb, int stride,
                                                            int ny, uint32_t nrows, Magic mny,
                                                            float2* __restrict__ X) {
  extern __shared__ __align__(16) float2 s_g[];  // twiddles, then rb rows
  const int n = p.n, nh = n / 2 + 1, rb = 1 << lrb;
  float2* tw = s_g;
  float2* buf = s_g + gen_tw_size(p);
  gen_twiddles(tw, (double2*)buf, p);
  const GPass p0 = p.p[0];
  const uint32_t tr = 2u << lrb, ntiles = (nrows + tr - 1) / tr;
  // the first pass's counts of a tile (rows 2p and 2p + 1), loaded while the tile before is
  // transformed and written
  DT ca[kGenXEpt], cb[kGenXEpt];
  auto load = [&](uint32_t tile) {
    gen_radix(p0.r, [&](auto rc) {
      constexpr int R = decltype(rc)::value;
      gen_each<R, kGenXEpt, kGenXThreads>(gen_tid(), p0, rb, [&](int b, int row, int j) {
        const uint32_t r = min(tile * tr + 2 * row, nrows - 2);  // nrows is even; rows past it are not written
        const DT* src = D + (int64_t)r * n + j;
#pragma unroll
        for (int q = 0; q < R; ++q) {
          ca[b * R + q] = src[q * p0.m];
          cb[b * R + q] = src[n + q * p0.m];
        }
      });
    });
  };
  if (blockIdx.x < ntiles) load(blockIdx.x);
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint32_t r0 = tile * tr;
    gen_radix(p0.r, [&](auto rc) {
      constexpr int R = decltype(rc)::value;
      const int tid = gen_tid();
      float2 v[R * gen_per_thread(R, kGenXEpt)];
#pragma unroll
      for (int e = 0; e < R * gen_per_thread(R, kGenXEpt); ++e) v[e] = make_float2((float)ca[e], (float)cb[e]);
      gen_compute<R, kGenXEpt, kGenXThreads, false>(tid, v, tw, p0, rb);
      gen_write<R, kGenXEpt, kGenXThreads>(tid, v, buf, stride, p0, rb);
    });
    if (tile + gridDim.x < ntiles) load(tile + gridDim.x);
    __syncthreads();
    for (int s = 1; s < p.np; ++s) {
      const GPass ps = p.p[s];
      gen_pass<kGenXEpt, kGenXThreads, true>(buf, stride, tw, ps, rb);
    }
    // z = a + i b of rows (2p, 2p+1): A(m) = (z(m) + conj z(-m))/2, B(m) = (z(m) - conj z(-m))/(2i)
    const int pr = (int)threadIdx.x & (rb - 1);
    const uint32_t r = r0 + 2 * pr;
    if (r < nrows) {
      const uint32_t kd = magic_div(r, mny), ry = r - kd * ny;
      float2* out = X + (int64_t)kd * nh * ny + ry;
      const float2* z = buf + pr * stride;
      for (int m = (int)threadIdx.x >> lrb; m < nh; m += kGenXThreads >> lrb) {
        const float2 u = z[m], w = cconj(z[m ? n - m : 0]);
        const float2 va = cscale(cadd(u, w), 0.5f), vb = cscale(cmul_mi(csub(u, w)), 0.5f);
        *(float4*)(out + (int64_t)m * ny) = make_float4(va.x, va.y, vb.x, vb.y);
      }
    }
    __syncthreads();
  }
}

int gen_x_rows(const GPlan& p, int64_t nrows, int& stride) {
  // row pairs per workgroup: 64 KB of rows at most where that is more than one pair; past 8 (runs of
  // 128 bytes) only while every compute unit still gets two workgroups
  const int most = gen_max_rows(p, kGenXThreads, kGenXEpt);
  if (most < 1) return -1;
  int lrb = 0;
  while ((2 << lrb) <= most && (2 << lrb) * p.len <= 8704 &&
         ((2 << lrb) <= 8 || nrows >= (4ll << lrb) * 512))
    ++lrb;
  // the row stride: 1 / rb of the banks apart modulo the 32 of 8 bytes, so that the rb rows of one
  // frequency, read together by the split, lie in different banks
  stride = p.len;
  const int step = 32 >> lrb ? 32 >> lrb : 1;
  while (lrb && (stride & 31) != step) ++stride;
  return lrb;
}

int launch_gen_x(int n, const void* D, int d_bits, int ny, int64_t nrows, float2* X, hipStream_t stream) {
  GPlan p;
  if (!gen_plan(n, p) || (ny & 1) || (nrows & 1) || nrows <= 0 || nrows >= (1ll << 31)) return STEM_EINVAL;
  int stride;
  const int lrb = gen_x_rows(p, nrows, stride);
  if (lrb < 0) return STEM_EINVAL;
  STEM_TRACE("xstage_fft", stream);
  const size_t lds = gen_lds(p, 1 << lrb, stride);
  auto go = [&](auto dt) {
    using DT = decltype(dt);
    const int64_t tiles = (nrows + (2 << lrb) - 1) / (2 << lrb);
    const int res = resident_blocks((const void*)k_grow_x<DT>, kGenXThreads, lds);
    const int64_t cap = res > 0 ? res : 512;
    hipLaunchKernelGGL(k_grow_x<DT>, dim3((unsigned)(tiles < cap ? tiles : cap)), dim3(kGenXThreads), lds, stream,
                       (const DT*)D, p, lrb, stride, ny, (uint32_t)nrows, make_magic((uint32_t)ny), X);
  };
  if (d_bits == 8) go(uint8_t{});
  else go(uint16_t{});
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

int launch_row_fft(int n, bool inverse, RowIn in, RowOut out, const RowFftArgs& a, hipStream_t stream) {
  if (a.nrows <= 0) return STEM_OK;
  STEM_TRACE(a.tag ? a.tag : "row_fft", stream);
  if (in == IN_U8 || in == IN_U16 || out == OUT_X) return STEM_EINVAL;
  if (!fast_length(n)) return launch_generic(n, inverse, in, out, a, stream);
  switch (n) {
    case 32: launch_n<32>(inverse, a, in, out, stream); break;
    case 64: launch_n<64>(inverse, a, in, out, stream); break;
    case 128: launch_n<128>(inverse, a, in, out, stream); break;
    case 256: launch_n<256>(inverse, a, in, out, stream); break;
    case 512: launch_n<512>(inverse, a, in, out, stream); break;
    case 1024: launch_n<1024>(inverse, a, in, out, stream); break;
    default: return STEM_EINVAL;
  }
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

// ---------------------------------------------------------------------------------------------
// The summed input of an IN_C64_SUM pass by itself, for many partials: one element per lane, its
// partials added in order (as the pass adds them, bit for bit) with kPartLoads of them in flight.  In the
// pass itself a wave adds the partials of 16 elements per lane, and a short transform leaves only a
// few waves to do so: 64 x 64 (one workgroup, 176 partials) 86 us, 256 x 256 (33) 44 us, 512 x 512 (10
// segments) 24 us, against 9 to 10 us here and 6 to 9 us for the pass without them.

constexpr int kPartLoads = 16;

template <bool SEG>
__global__ void __launch_bounds__(64) k_part_sum(RowFftArgs a, int n) {
  const int lane = threadIdx.x;
  if (a.stats && blockIdx.x == gridDim.x - 1) {
    // the last workgroup, which no element has, adds the fused sums' per-wave counters
    unsigned long long c = 0, l = 0;
    for (int64_t i0 = lane; i0 < a.nwcnt; i0 += 64 * kPartLoads) {
      unsigned long long w[kPartLoads];
#pragma unroll
      for (int u = 0; u < kPartLoads; ++u) w[u] = i0 + 64 * u < a.nwcnt ? a.wcnt[i0 + 64 * u] : 0ull;
#pragma unroll
      for (int u = 0; u < kPartLoads; ++u) {
        c += w[u] & ((1ull << 40) - 1);
        l += w[u] >> 40;
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      c += __shfl_xor(c, off);
      l += __shfl_xor(l, off);
    }
    if (lane == 0) {
      a.stats[0] = c;
      a.stats[1] = SEG ? (unsigned long long)a.part_seg[a.nrows] : (unsigned long long)a.stats_groups;
      a.stats[2] = 8ull * l;
      a.stats[3] = (unsigned long long)a.stats_chunks;
      if (a.ready_out) *a.ready_out = a.ready_val;
    }
    return;
  }
  const int64_t el = (int64_t)blockIdx.x * 64 + lane, total = a.nrows * n;
  if (el >= total) return;
  const float2* src = a.in_c + el;
  int64_t step = a.part_stride;
  int count = a.nparts;
  if constexpr (SEG) {
    const int64_t r = el / n;
    const int64_t s0 = min(max(a.part_seg[r], (int64_t)0), a.part_seg_rows);
    count = (int)(min(max(a.part_seg[r + 1], s0), a.part_seg_rows) - s0);
    src = a.in_c + s0 * n + (el - r * n);
    step = n;
  }
  float2 x = make_float2(0.f, 0.f);
  for (int q = 0; q < count; q += kPartLoads) {
    float2 t[kPartLoads];
#pragma unroll
    for (int u = 0; u < kPartLoads; ++u) t[u] = q + u < count ? src[(q + u) * step] : make_float2(0.f, 0.f);
#pragma unroll
    for (int u = 0; u < kPartLoads; ++u) x = cadd(x, t[u]);
  }
  if (a.norm_cnt) {
    const int32_t c = a.norm_cnt[el];
    x = c > 0 ? make_float2(x.x / (float)c, x.y / (float)c) : make_float2(0.f, 0.f);
  }
  a.sum_out[el] = x;
}

int launch_part_sum(int n, const RowFftArgs& a, hipStream_t stream) {
  if (!a.sum_out || a.nrows <= 0) return STEM_EINVAL;
  STEM_TRACE("part_sum", stream);
  const dim3 grid((unsigned)((a.nrows * n + 63) / 64 + (a.stats ? 1 : 0))), blk(64);
  if (a.part_seg) hipLaunchKernelGGL(k_part_sum<true>, grid, blk, 0, stream, a, n);
  else hipLaunchKernelGGL(k_part_sum<false>, grid, blk, 0, stream, a, n);
  STEM_LAUNCH_CHECK();
  return STEM_OK;
}

// ---------------------------------------------------------------------------------------------
// DPC: per-frequency recurrence (Sec. V).  C = FFT2(gx + i gy) row-major [my][mx]; the two real
// spectra are Gx = (C(q) + conj C(-q))/2, Gy = (C(q) - conj C(-q))/(2i).  With D = 2 pi i q and
// d = lam1 + |2 pi q|^2 + lam2 |2 pi q|^4:  Phi <- Phi + mu conj(D).(G - D Phi)/d, L times, in
// double; q = 0 and the Nyquist row/column are held at zero.

// The descent of one frequency from Phi = 0, in closed form: with b = conj(D).G and r = 1 - mu q^2/d a step
// is Phi <- r Phi + (mu/d) b, so L steps give (mu/d) b S with S = 1 + r + ... + r^(L-1), L dependent
// multiply-adds instead of 4 L with 12 operations each (1024 x 1024, L = 10: the column pass 18.4 us instead
// of 21.4 us).
__device__ __forceinline__ float2 dpc_descend(float2 gx, float2 gy, double qx, double qy, double mu, double lam1,
                                              double lam2, int n_iter, bool live) {
  const double q2 = qx * qx + qy * qy;
  const double d = lam1 + q2 + lam2 * q2 * q2;
  if (!live || d == 0.0 || n_iter <= 0) return make_float2(0.f, 0.f);
  const double md = mu / d, r = 1.0 - md * q2;
  double s = 1.0;
  for (int l = 1; l < n_iter; ++l) s = s * r + 1.0;
  s *= md;
  // a zero b stays at Phi = 0 in every step, also where the steps diverge and S is not finite
  const double br = qx * (double)gx.y + qy * (double)gy.y, bi = -(qx * (double)gx.x + qy * (double)gy.x);
  return make_float2(br == 0.0 ? 0.f : (float)(s * br), bi == 0.0 ? 0.f : (float)(s * bi));
}

// ---------------------------------------------------------------------------------------------
// DPC integration in three passes over the packed gradient z = gx + i gy (Sec. V):
//  k_dpc_rows  rows ry: FFT along rx, split into the half spectra Gx, Gy along x (z(m) and
//              conj z(-m)), written transposed [mx][ry] for mx in [0, Nx/2];
//  k_dpc_cols  rows mx: FFT of both along ry, the per-frequency gradient descent (no mirror
//              element needed: Gx and Gy are separate), inverse FFT along my, written
//              transposed [ry][mx] (half spectrum along x);
//  then k_row_fft (IN_HALF_C64) rows ry: inverse along mx of the Hermitian row, real part / F.

template <int N, int W>
__global__ void __launch_bounds__(64 * W) k_dpc_rows(const double* __restrict__ c64, const float* __restrict__ c32,
                                                   int64_t plane, int ny, float g, float2* __restrict__ Ax,
                                                   float2* __restrict__ Ay) {
  constexpr int kThreads = 64 * W;
  constexpr int B = 1024 / N, TR = W * B, NH = N / 2 + 1;
  __shared__ float2 s_tw[1024];
  __shared__ float2 s_buf[W * kWaveStride];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  fill_twiddles(s_tw, threadIdx.x, kThreads);
  __syncthreads();
  float2* buf = s_buf + wave * kWaveStride;
  const int ntiles = (ny + TR - 1) / TR;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int r0 = tile * TR + wave * B;
    float2 v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      int b, n;
      fft_in_index<N>(lane, i, b, n);
      const int r = r0 + b;
      float2 x = make_float2(0.f, 0.f);
      if (r < ny) {
        const int64_t e = (int64_t)r * N + n;
        x = c64 ? make_float2((float)(c64[e] * (double)g), (float)(c64[plane + e] * (double)g))
                : make_float2(c32[e] * g, c32[plane + e] * g);
      }
      v[i] = x;
    }
    wave_fft<N>(v, buf, s_tw, lane);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      int b, m;
      fft_out_index<N>(lane, i, b, m);
      buf[fft_pad(b * N + m)] = v[i];
    }
    __syncthreads();
    for (int u = threadIdx.x; u < TR * NH; u += kThreads) {
      const int m = u / TR, rl = u % TR;
      const int w = rl / B, b = rl % B;
      const int r = tile * TR + rl;
      if (r < ny) {
        const float2* wb = s_buf + w * kWaveStride;
        const float2 z = wb[fft_pad(b * N + m)];
        const float2 zc = cconj(wb[fft_pad(b * N + ((N - m) & (N - 1)))]);
        Ax[(int64_t)m * ny + r] = cscale(cadd(z, zc), 0.5f);
        Ay[(int64_t)m * ny + r] = cscale(cmul_mi(csub(z, zc)), 0.5f);
      }
    }
    __syncthreads();
  }
}

template <int N, int W>
__global__ void __launch_bounds__(64 * W) k_dpc_cols(const float2* __restrict__ Ax, const float2* __restrict__ Ay,
                                                   int nx, double step, double mu, double lam1, double lam2,
                                                   int n_iter, float2* __restrict__ Q) {
  constexpr int kThreads = 64 * W;
  constexpr int B = 1024 / N, TR = W * B;
  __shared__ float2 s_tw[1024];
  __shared__ float2 s_buf[W * kWaveStride];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  fill_twiddles(s_tw, threadIdx.x, kThreads);
  __syncthreads();
  float2* buf = s_buf + wave * kWaveStride;
  const int nh = nx / 2 + 1;
  const int ntiles = (nh + TR - 1) / TR;
  const double two_pi = 6.283185307179586476925286766559;
  const double dqx = two_pi / ((double)nx * step), dqy = two_pi / ((double)N * step);
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int r0 = tile * TR + wave * B;  // rows are frequencies mx
    float2 vx[16], vy[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      int b, n;
      fft_in_index<N>(lane, i, b, n);
      const int r = r0 + b;
      vx[i] = r < nh ? Ax[(int64_t)r * N + n] : make_float2(0.f, 0.f);
      vy[i] = r < nh ? Ay[(int64_t)r * N + n] : make_float2(0.f, 0.f);
    }
    wave_fft<N>(vx, buf, s_tw, lane);
    wave_fft<N>(vy, buf, s_tw, lane);
    // gradient descent per frequency (my, mx); the result goes to LDS in natural order
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      int b, my;
      fft_out_index<N>(lane, i, b, my);
      const int mx = r0 + b;
      const int sy = my < (N + 1) / 2 ? my : my - N;
      const int sx = mx < (nx + 1) / 2 ? mx : mx - nx;
      const float2 ph = dpc_descend(vx[i], vy[i], (double)sx * dqx, (double)sy * dqy, mu, lam1, lam2, n_iter,
                                    !(my == 0 && mx == 0) && my != N / 2 && mx != nx / 2 && mx < nh);
      buf[fft_pad(b * N + my)] = ph;
    }
    wave_lds_sync();
    // inverse along my: conj, forward transform, conj
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      int b, n;
      fft_in_index<N>(lane, i, b, n);
      vx[i] = cconj(buf[fft_pad(b * N + n)]);
    }
    wave_lds_sync();
    wave_fft<N>(vx, buf, s_tw, lane);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      int b, m;
      fft_out_index<N>(lane, i, b, m);
      buf[fft_pad(b * N + m)] = cconj(vx[i]);
    }
    __syncthreads();
    // transposed write: Q[ry][mx], runs of TR frequencies mx
    for (int u = threadIdx.x; u < TR * N; u += kThreads) {
      const int m = u / TR, rl = u % TR;
      const int w = rl / B, b = rl % B;
      const int r = tile * TR + rl;
      if (r < nh) Q[(int64_t)m * nh + r] = s_buf[w * kWaveStride + fft_pad(b * N + m)];
    }
    __syncthreads();
  }
}

template <int N>
static void launch_dpc_rows(const double* c64, const float* c32, int64_t plane, int ny, float g, float2* Ax,
                            float2* Ay, hipStream_t s) {
  constexpr int W = 4;
  const int tiles = (ny + W * (1024 / N) - 1) / (W * (1024 / N));
  hipLaunchKernelGGL((k_dpc_rows<N, W>), dim3((unsigned)tiles), dim3(64 * W), 0, s, c64, c32, plane, ny, g, Ax, Ay);
}

template <int N>
static void launch_dpc_cols(const float2* Ax, const float2* Ay, int nx, double step, const stem_dpc& p, float2* Q,
                            hipStream_t s) {
  constexpr int W = 4;
  const int nh = nx / 2 + 1;
  const int tiles = (nh + W * (1024 / N) - 1) / (W * (1024 / N));
  hipLaunchKernelGGL((k_dpc_cols<N, W>), dim3((unsigned)tiles), dim3(64 * W), 0, s, Ax, Ay, nx, step, p.mu, p.lam1,
                     p.lam2, p.n_iter, Q);
}

// the three DPC passes for power-of-two lengths in [32, 1024]
static int launch_dpc(const double* c64, const float* c32, int64_t F, int ny, int nx, float g, double step,
                      const stem_dpc& p, float2* Ax, float2* Ay, float2* Q, float* phase, hipStream_t s) {
  {
    STEM_TRACE("dpc_rows", s);
    switch (nx) {
      case 32: launch_dpc_rows<32>(c64, c32, F, ny, g, Ax, Ay, s); break;
      case 64: launch_dpc_rows<64>(c64, c32, F, ny, g, Ax, Ay, s); break;
      case 128: launch_dpc_rows<128>(c64, c32, F, ny, g, Ax, Ay, s); break;
      case 256: launch_dpc_rows<256>(c64, c32, F, ny, g, Ax, Ay, s); break;
      case 512: launch_dpc_rows<512>(c64, c32, F, ny, g, Ax, Ay, s); break;
      case 1024: launch_dpc_rows<1024>(c64, c32, F, ny, g, Ax, Ay, s); break;
      default: return STEM_EINVAL;
    }
    STEM_LAUNCH_CHECK();
  }
  {
    STEM_TRACE("dpc_cols", s);
    switch (ny) {
      case 32: launch_dpc_cols<32>(Ax, Ay, nx, step, p, Q, s); break;
      case 64: launch_dpc_cols<64>(Ax, Ay, nx, step, p, Q, s); break;
      case 128: launch_dpc_cols<128>(Ax, Ay, nx, step, p, Q, s); break;
      case 256: launch_dpc_cols<256>(Ax, Ay, nx, step, p, Q, s); break;
      case 512: launch_dpc_cols<512>(Ax, Ay, nx, step, p, Q, s); break;
      case 1024: launch_dpc_cols<1024>(Ax, Ay, nx, step, p, Q, s); break;
      default: return STEM_EINVAL;
    }
    STEM_LAUNCH_CHECK();
  }
  // inverse along mx of the Hermitian rows, real part / F -> phase[ry][rx]
  RowFftArgs a{};
  a.nrows = ny;
  a.in_c = Q;
  a.out_f = phase;
  a.osc = make_float2((float)(1.0 / (double)F), 0.f);
  a.tag = "dpc_fft";
  return launch_row_fft(nx, true, IN_HALF_C64, OUT_ROW_RE, a, s);
}

// ---------------------------------------------------------------------------------------------
// DPC for the other scan lengths, in five passes of the generic FFT and one per-frequency pass:
// rows ry of z = g (COM_x + i COM_y) transformed along rx and written transposed [mx][ry]; rows mx
// transformed along ry in place (C = FFT2 z, column-major [mx][my]); the descent per frequency from
// Gx = (C(q) + conj C(-q))/2 and Gy = (C(q) - conj C(-q))/(2i) into Phi; the inverse along my,
// written transposed [ry][mx]; the inverse along mx, real part / F.

__global__ void __launch_bounds__(256) k_dpc_descent(const float2* __restrict__ C, int ny, int nx, double dqx,
                                                     double dqy, double mu, double lam1, double lam2, int n_iter,
                                                     float2* __restrict__ Phi) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (int64_t)ny * nx) return;
  const int mx = (int)(q / ny), my = (int)(q % ny);
  const float2 c = C[q];
  const float2 cm = cconj(C[(int64_t)((nx - mx) % nx) * ny + (ny - my) % ny]);
  const int sy = my < (ny + 1) / 2 ? my : my - ny;
  const int sx = mx < (nx + 1) / 2 ? mx : mx - nx;
  // Gx = (c + cm)/2, Gy = (c - cm)/(2i)
  const float2 gx = make_float2(0.5f * (c.x + cm.x), 0.5f * (c.y + cm.y));
  const float2 gy = make_float2(0.5f * (c.y - cm.y), -0.5f * (c.x - cm.x));
  Phi[q] = dpc_descend(gx, gy, (double)sx * dqx, (double)sy * dqy, mu, lam1, lam2, n_iter,
                       !(my == 0 && mx == 0) && 2 * my != ny && 2 * mx != nx);
}

static int launch_dpc_generic(const double* c64, const float* c32, int64_t F, int ny, int nx, float g, double step,
                              const stem_dpc& p, float2* A, float2* B, float* phase, hipStream_t s) {
  RowFftArgs a{};
  a.nrows = ny;
  if (c64) {
    a.in_d0 = c64;
    a.in_d1 = c64 + F;
  } else {
    a.in_f0 = c32;
    a.in_f1 = c32 + F;
  }
  a.s0 = a.s1 = g;
  a.out_c = A;
  a.out_stride = ny;
  a.osc = make_float2(1.f, 0.f);
  a.tag = "dpc_fft";
  int st = launch_row_fft(nx, false, c64 ? IN_F64_PAIR : IN_F32_PAIR, OUT_T_C64, a, s);
  if (st) return st;
  a = RowFftArgs{};
  a.nrows = nx;
  a.in_c = A;
  a.out_c = A;
  a.osc = make_float2(1.f, 0.f);
  a.tag = "dpc_fft";
  if ((st = launch_row_fft(ny, false, IN_C64, OUT_ROW_C64, a, s))) return st;
  {
    STEM_TRACE("dpc_descent", s);
    const double two_pi = 6.283185307179586476925286766559;
    hipLaunchKernelGGL(k_dpc_descent, dim3((unsigned)((F + 255) / 256)), dim3(256), 0, s, A, ny, nx,
                       two_pi / ((double)nx * step), two_pi / ((double)ny * step), p.mu, p.lam1, p.lam2, p.n_iter, B);
    STEM_LAUNCH_CHECK();
  }
  a = RowFftArgs{};
  a.nrows = nx;
  a.in_c = B;
  a.out_c = A;
  a.out_stride = nx;
  a.osc = make_float2(1.f, 0.f);
  a.tag = "dpc_fft";
  if ((st = launch_row_fft(ny, true, IN_C64, OUT_T_C64, a, s))) return st;
  a = RowFftArgs{};
  a.nrows = ny;
  a.in_c = A;
  a.out_f = phase;
  a.osc = make_float2((float)(1.0 / (double)F), 0.f);
  a.tag = "dpc_fft";
  return launch_row_fft(nx, true, IN_C64, OUT_ROW_RE, a, s);
}

}  // namespace stem

// ---------------------------------------------------------------------------------------------
// C ABI

using namespace stem;

extern "C" size_t com_dpc_workspace_bytes(const stem_scan* scan) {
  if (!scan || scan->ny <= 0 || scan->nx <= 0) return 0;
  if (fast_length(scan->ny) && fast_length(scan->nx))
    // the half spectra Gx, Gy along x and the half-spectrum result, (Nx/2+1) Ny complex64 each
    return 3 * align256((size_t)scan->ny * (scan->nx / 2 + 1) * sizeof(float2));
  // the other lengths: the full transform of z and the descent's result, F complex64 each
  return 2 * align256((size_t)scan->ny * scan->nx * sizeof(float2));
}

static int run_com_dpc(const int32_t* d_idx, const int64_t* d_off, int64_t frame0, int64_t n_frames,
                       const stem_det* det, const stem_scan* scan, const stem_optics* optics, const stem_dpc* dpc,
                       double* d_com64, float* d_com32, int32_t* d_counts, float* d_phase, void* ws,
                       size_t ws_bytes, int32_t* d_status, void* stream_) {
  if (!d_idx || !d_off || !det || !scan) return STEM_EINVAL;
  if (det->W <= 0 || det->H <= 0 || (int64_t)det->W * det->H >= (1ll << 31)) return STEM_EINVAL;
  if (scan->ny <= 0 || scan->nx <= 0) return STEM_EINVAL;
  const int64_t F = (int64_t)scan->ny * scan->nx;
  if (frame0 < 0 || n_frames < 0 || frame0 + n_frames > F) return STEM_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  if (d_phase) {
    if (!optics || !dpc || (!d_com64 && !d_com32)) return STEM_EINVAL;
    if (!scan_length_ok(scan->ny) || !scan_length_ok(scan->nx)) return STEM_EINVAL;
    if (!(scan->step > 0) || !(optics->dk > 0) || dpc->n_iter < 0) return STEM_EINVAL;
    if (!ws || ws_bytes < com_dpc_workspace_bytes(scan) || ((uintptr_t)ws & 255)) return STEM_EWORKSPACE;
  }
  int st = launch_com(d_idx, d_off, frame0, n_frames, *det, F, d_com64, d_com32, d_counts, d_status, stream);
  if (st != STEM_OK || !d_phase) return st;

  const int ny = scan->ny, nx = scan->nx;
  const float g = (float)(2.0 * 3.14159265358979323846 * optics->dk);
  if (!fast_length(ny) || !fast_length(nx)) {
    float2* A = (float2*)ws;
    float2* B = (float2*)((char*)ws + align256((size_t)F * sizeof(float2)));
    return launch_dpc_generic(d_com64, d_com64 ? nullptr : d_com32, F, ny, nx, g, scan->step, *dpc, A, B, d_phase,
                              stream);
  }
  const size_t half = align256((size_t)ny * (nx / 2 + 1) * sizeof(float2));
  float2* Ax = (float2*)ws;
  float2* Ay = (float2*)((char*)ws + half);
  float2* Q = (float2*)((char*)ws + 2 * half);
  return launch_dpc(d_com64, d_com64 ? nullptr : d_com32, F, ny, nx, g, scan->step, *dpc, Ax, Ay, Q, d_phase, stream);
}

extern "C" int com_dpc(const int32_t* d_idx, const int64_t* d_off, int64_t frame0, int64_t n_frames,
                       const stem_det* det, const stem_scan* scan, const stem_optics* optics,
                       const stem_dpc* dpc, double* d_com64, float* d_com32, int32_t* d_counts,
                       float* d_phase, void* ws, size_t ws_bytes, int32_t* d_status, void* stream_) {
  return run_com_dpc(d_idx, d_off, frame0, n_frames, det, scan, optics, dpc, d_com64, d_com32, d_counts, d_phase, ws,
                     ws_bytes, d_status, stream_);
}

// ---------------------------------------------------------------------------------------------
// com_dpc without a caller workspace: the DPC integration's half-spectrum planes live in a
// file-scope device array (one copy per GPU, held until the process ends).  In host code the
// array's name is not a device address: its address on each device is looked up once, with that
// device current, and only that pointer is passed to kernels.

namespace {

constexpr size_t kNoAllocScratchBytes = (size_t)16 << 20;
__device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// this device's copy of `scratch`, looked up on its first use (nullptr if the lookup fails)
void* scratch_on_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

}  // namespace

extern "C" size_t com_dpc_noalloc_max_workspace(void) { return kNoAllocScratchBytes; }

extern "C" int com_dpc_noalloc(const int32_t* d_idx, const int64_t* d_off, int64_t frame0, int64_t n_frames,
                               const stem_det* det, const stem_scan* scan, const stem_optics* optics,
                               const stem_dpc* dpc, double* d_com64, float* d_com32, int32_t* d_counts,
                               float* d_phase, int32_t* d_status, void* stream_) {
  void* ws = nullptr;
  if (d_phase) {
    if (!scan) return STEM_EINVAL;
    if (com_dpc_workspace_bytes(scan) > kNoAllocScratchBytes) return STEM_EWORKSPACE;
    ws = scratch_on_current_device();
    if (!ws) return STEM_EHIP;
  }
  return run_com_dpc(d_idx, d_off, frame0, n_frames, det, scan, optics, dpc, d_com64, d_com32, d_counts, d_phase, ws,
                     d_phase ? kNoAllocScratchBytes : 0, d_status, stream_);
}

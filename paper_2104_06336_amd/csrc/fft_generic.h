// Mixed-radix FFT of any even length N = 2^a 3^b 5^c up to kGenMax, for the scan sizes the wavefront
// FFT of fft_wave.h does not take (not a power of two, or longer than 1024).
//
// A workgroup transforms RB rows at once in LDS with a Stockham autosort FFT: pass s of radix R, with
// Ns the product of the earlier radices and m = N/R, takes butterfly j (0 <= j < m) from elements
// j + q m (q < R), multiplies element q by w^(q (j mod Ns)) with w = exp(-2 pi i / (Ns R)), applies the
// length-R DFT and writes element q to (j div Ns) Ns R + (j mod Ns) + q Ns.  Every thread reads all
// its butterflies' inputs before the workgroup barrier and writes after it, so one LDS buffer serves
// each pass in place.
//
// What bounds it is LDS traffic, index arithmetic and barriers, all per pass, so the plan takes the
// fewest passes it can: radices up to 16 (1000 = 10.10.10, 96 = 8.12, 2000 = 5.5.8.10), the composite
// ones in registers (products of coprime lengths by the prime-factor map, without twiddles).  The
// twiddles lie in LDS per pass in the order the butterflies read them ([q - 1][j mod Ns], N - R0
// entries in all), the quotients by m and Ns are multiply-high by constants of the plan.  Against radices
// 4, 2, 3, 5 taken one by one with a table of W_N^t (an FP64 sincospi per entry and workgroup) and
// integer divisions, 1000 rows of 1000 take 23 us instead of 30 us (one MI355X), 160 rows of 96 6.7 us
// instead of 23 us.
#pragma once

#include "common.h"
#include "fft_wave.h"

namespace stem {

constexpr int kGenMax = 4096;     // longest transform
constexpr int kGenThreads = 256;  // threads of a generic-FFT workgroup of the row passes
constexpr int kGenMaxPasses = 6;

// One pass: radix r, m = n/r, ns the product of the earlier radices, off the pass's first twiddle,
// step = n/(ns r); mm and mns divide by m and ns (gdiv).  LDS layouts: the pass reads element i of a row
// at i + (i div ns) rp and writes it at i + (i div (ns r)) wp (the next pass's rp), so that the element of
// q is a constant away from that of q - 1 on both sides (rq = m + (m div ns) rp apart read, ns written).
struct GPass {
  int32_t r, m, ns, off, step, rp, rq, wp;
  uint32_t mm, mns;
};

struct GPlan {
  int32_t n;
  int32_t np;
  int32_t ntw;  // twiddles of the passes after the first: n - r0
  int32_t len;  // LDS elements of a row in its longest layout
  uint32_t mn;  // divides by n
  GPass p[kGenMaxPasses];
};

// x / d for 0 <= x < 2^17, 1 <= d <= 4096: with mag = ceil(2^32 / d), mag d - 2^32 < d and x d < 2^29,
// so the error x (mag d - 2^32) / (d 2^32) stays below 1/d.  d = 1 has no 32-bit mag (0 stands for it).
inline uint32_t gmagic(int d) { return d == 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d); }
__device__ __forceinline__ int gdiv(int x, uint32_t mag) { return mag ? (int)__umulhi((uint32_t)x, mag) : x; }

// The plan of n = 2^a 3^b 5^c, 4 <= n <= kGenMax: radices ascending, the fewest passes (at least two) and
// then the smallest sum; the largest radix is the last pass's, whose butterflies are the fewest, at
// most one per thread in the fused sum.  False for other lengths.  A length's plan is formed once and
// kept (about a hundred lengths exist).
bool gen_plan(int n, GPlan& p);

// Butterflies of radix r a thread takes in a pass with ept registers, and the rows of a workgroup of
// t threads that respect it in every pass.
__host__ __device__ constexpr int gen_per_thread(int r, int ept) { return ept / r > 1 ? ept / r : 1; }
inline int gen_max_rows(const GPlan& p, int threads, int ept) {
  int rb = kGenMax;
  for (int s = 0; s < p.np; ++s) {
    const int k = threads * gen_per_thread(p.p[s].r, ept) / p.p[s].m;
    rb = k < rb ? k : rb;
  }
  return rb;
}

// Rows a workgroup of the row passes takes of nrows, and the binary logarithm of the row pairs one of the
// row transform of counts takes, with its LDS row stride (-1: none).
int gen_fft_rows(const GPlan& p, int64_t nrows);
int gen_x_rows(const GPlan& p, int64_t nrows, int& stride);

// LDS of a workgroup in float2: the twiddles (an even number of entries, so that what follows is
// 16-byte aligned), then the rows (at least the 128 double2 that gen_twiddles works in)
__host__ __device__ inline int gen_tw_size(const GPlan& p) { return (p.ntw + 1) & ~1; }
inline size_t gen_lds(const GPlan& p, int rows, int stride) {
  const size_t b = (size_t)rows * stride;
  return ((size_t)gen_tw_size(p) + (b < 256 ? 256 : b)) * sizeof(float2);
}

// The passes' twiddles, tw[off + (q - 1) ns + k] = W_N^(q k step), FP64 rounded to FP32: W_N^t is the
// FP64 product of W_N^(t mod 64) and W_N^(64 (t div 64)), 128 sincospi in all instead of one per
// entry.  scratch: 128 double2 of LDS, free afterwards.  Every thread of the workgroup takes part (at
// least 128); it ends with a barrier.
__device__ __forceinline__ void gen_twiddles(float2* tw, double2* scratch, const GPlan& p) {
  if (threadIdx.x < 128) {
    const int t = threadIdx.x < 64 ? threadIdx.x : 64 * (threadIdx.x - 64);
    double s, c;
    sincospi(2.0 * (double)t / (double)p.n, &s, &c);
    scratch[threadIdx.x] = make_double2(c, -s);
  }
  __syncthreads();
  for (int s = 1; s < p.np; ++s) {
    const GPass& g = p.p[s];
    const int ne = g.ns * (g.r - 1);
    for (int e = threadIdx.x; e < ne; e += blockDim.x) {
      const int q1 = gdiv(e, g.mns), k = e - q1 * g.ns;
      const int t = (q1 + 1) * k * g.step;  // below n
      const double2 a = scratch[t & 63], b = scratch[64 + (t >> 6)];
      tw[g.off + e] = make_float2((float)(a.x * b.x - a.y * b.y), (float)(a.x * b.y + a.y * b.x));
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------------------------
// length-R DFTs in registers (forward sign), natural order in and out

// X_k = sum_n x_n exp(-2 pi i n k / 3): with s = x1 + x2, d = x1 - x2,
// X_0 = x0 + s, X_{1,2} = x0 - s/2 -/+ i (sqrt(3)/2) d
__device__ __forceinline__ void gdft3(float2* v) {
  constexpr float h = 0.86602540378443864676f;  // sqrt(3)/2
  const float2 s = cadd(v[1], v[2]), d = csub(v[1], v[2]);
  const float2 m = make_float2(v[0].x - 0.5f * s.x, v[0].y - 0.5f * s.y);
  const float2 r = make_float2(h * d.y, -h * d.x);  // -i (sqrt(3)/2) d
  v[0] = cadd(v[0], s);
  v[1] = cadd(m, r);
  v[2] = csub(m, r);
}

// length 5 from its definition, with cos and sin of 2 pi/5 and 4 pi/5: pairs (x1, x4) and (x2, x3)
// give X_k = x0 + c_k1 (x1 + x4) + c_k2 (x2 + x3) - i (s_k1 (x1 - x4) + s_k2 (x2 - x3))
__device__ __forceinline__ void gdft5(float2* v) {
  constexpr float c1 = 0.30901699437494742410f, c2 = -0.80901699437494742410f;  // cos 2pi/5, cos 4pi/5
  constexpr float s1 = 0.95105651629515357212f, s2 = 0.58778525229247312917f;   // sin 2pi/5, sin 4pi/5
  const float2 a1 = cadd(v[1], v[4]), b1 = csub(v[1], v[4]);
  const float2 a2 = cadd(v[2], v[3]), b2 = csub(v[2], v[3]);
  const float2 x0 = v[0];
  const float2 p1 = make_float2(x0.x + c1 * a1.x + c2 * a2.x, x0.y + c1 * a1.y + c2 * a2.y);
  const float2 p2 = make_float2(x0.x + c2 * a1.x + c1 * a2.x, x0.y + c2 * a1.y + c1 * a2.y);
  const float2 q1 = make_float2(s1 * b1.x + s2 * b2.x, s1 * b1.y + s2 * b2.y);   // k = 1
  const float2 q2 = make_float2(s2 * b1.x - s1 * b2.x, s2 * b1.y - s1 * b2.y);   // k = 2
  v[0] = make_float2(x0.x + a1.x + a2.x, x0.y + a1.y + a2.y);
  v[1] = make_float2(p1.x + q1.y, p1.y - q1.x);  // p1 - i q1
  v[4] = make_float2(p1.x - q1.y, p1.y + q1.x);  // p1 + i q1
  v[2] = make_float2(p2.x + q2.y, p2.y - q2.x);
  v[3] = make_float2(p2.x - q2.y, p2.y + q2.x);
}

// length 9 = 3 x 3 (n = n1 + 3 n2, X[k2 + 3 k1]), the inner twiddles exp(-2 pi i n1 k2 / 9)
__device__ __forceinline__ void gdft9(float2* v) {
  const float2 w1 = make_float2(0.76604444311897803520f, -0.64278760968653932632f);   // 2 pi/9
  const float2 w2 = make_float2(0.17364817766693034885f, -0.98480775301220805937f);   // 4 pi/9
  const float2 w4 = make_float2(-0.93969262078590838405f, -0.34202014332566873304f);  // 8 pi/9
  float2 y[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
#pragma unroll
    for (int b = 0; b < 3; ++b) y[a][b] = v[a + 3 * b];
    gdft3(y[a]);
  }
  y[1][1] = cmul(y[1][1], w1);
  y[1][2] = cmul(y[1][2], w2);
  y[2][1] = cmul(y[2][1], w2);
  y[2][2] = cmul(y[2][2], w4);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    float2 c[3] = {y[0][k], y[1][k], y[2][k]};
    gdft3(c);
#pragma unroll
    for (int b = 0; b < 3; ++b) v[k + 3 * b] = c[b];
  }
}

template <int R>
__device__ __forceinline__ void gdft(float2* v);

// length A B, A and B coprime, by the prime-factor map: input n = (B a + A b) mod AB, output k with
// k mod A = ka and k mod B = kb; exp(-2 pi i n k / AB) = exp(-2 pi i a ka / A) exp(-2 pi i b kb / B)
template <int A, int B>
__device__ __forceinline__ void gdft_pfa(float2* v) {
  constexpr int N = A * B;
  float2 y[B][A];
#pragma unroll
  for (int b = 0; b < B; ++b) {
#pragma unroll
    for (int a = 0; a < A; ++a) y[b][a] = v[(B * a + A * b) % N];
    gdft<A>(y[b]);
  }
#pragma unroll
  for (int a = 0; a < A; ++a) {
    float2 c[B];
#pragma unroll
    for (int b = 0; b < B; ++b) c[b] = y[b][a];
    gdft<B>(c);
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (k % A == a) v[k] = c[k % B];
  }
}

template <int R>
__device__ __forceinline__ void gdft(float2* v) {
  if constexpr (R == 2) dft2(v);
  else if constexpr (R == 3) gdft3(v);
  else if constexpr (R == 4) dft4(v);
  else if constexpr (R == 5) gdft5(v);
  else if constexpr (R == 6) gdft_pfa<2, 3>(v);
  else if constexpr (R == 8) dft8(v);
  else if constexpr (R == 9) gdft9(v);
  else if constexpr (R == 10) gdft_pfa<2, 5>(v);
  else if constexpr (R == 12) gdft_pfa<4, 3>(v);
  else if constexpr (R == 15) gdft_pfa<3, 5>(v);
  else dft16(v);
}

// f(integral_constant R) for a plan's radix r <= MAX (the same for the whole workgroup)
template <int MAX = 16, typename F>
__device__ __forceinline__ void gen_radix(int r, F&& f) {
  switch (r) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 10: f(std::integral_constant<int, 10>{}); break;
    default:
      if constexpr (MAX >= 16) {
        if (r == 15) {
          f(std::integral_constant<int, 15>{});
          break;
        } else if (r == 16) {
          f(std::integral_constant<int, 16>{});
          break;
        }
      }
      f(std::integral_constant<int, 12>{});
      break;
  }
}

// ---------------------------------------------------------------------------------------------
// The parts of a pass of radix R over rb rows of the workgroup (T threads, EPT registers per thread):
// thread t takes butterflies g = t + T b < rb m, of row g / m, held at v[b R ..].

// The thread index, opaque to the compiler: a pass's index arithmetic depends on nothing that changes
// from tile to tile, and hoisted out of the tile loop (for every radix of the switch) it spills
// hundreds of registers.
__device__ __forceinline__ int gen_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

template <int R, int EPT, int T, typename F>
__device__ __forceinline__ void gen_each(int tid, const GPass& p, int rb, F&& f) {
  const int total = rb * p.m;
#pragma unroll
  for (int b = 0; b < gen_per_thread(R, EPT); ++b) {
    const int g = tid + b * T;
    if (g < total) {
      const int row = gdiv(g, p.mm);
      f(b, row, g - row * p.m);
    }
  }
}

// inputs from LDS
template <int R, int EPT, int T>
__device__ __forceinline__ void gen_read(int tid, float2* v, const float2* buf, int stride, const GPass& p, int rb) {
  gen_each<R, EPT, T>(tid, p, rb, [&](int b, int row, int j) {
    const float2* in = buf + row * stride + j + gdiv(j, p.mns) * p.rp;
#pragma unroll
    for (int q = 0; q < R; ++q) v[b * R + q] = in[q * p.rq];
  });
}

// twiddles (TW: not the first pass) and the length-R DFTs
template <int R, int EPT, int T, bool TW>
__device__ __forceinline__ void gen_compute(int tid, float2* v, const float2* tw, const GPass& p, int rb) {
  gen_each<R, EPT, T>(tid, p, rb, [&](int b, int, int j) {
    if constexpr (TW) {
      const float2* w = tw + p.off + (j - gdiv(j, p.mns) * p.ns);
#pragma unroll
      for (int q = 1; q < R; ++q) v[b * R + q] = cmul(v[b * R + q], w[(q - 1) * p.ns]);
    }
    gdft<R>(v + b * R);
  });
}

// outputs to LDS
template <int R, int EPT, int T>
__device__ __forceinline__ void gen_write(int tid, const float2* v, float2* buf, int stride, const GPass& p, int rb) {
  gen_each<R, EPT, T>(tid, p, rb, [&](int b, int row, int j) {
    // element (j div ns) ns R + j mod ns + q ns
    float2* out = buf + row * stride + j + gdiv(j, p.mns) * (p.ns * (R - 1) + p.wp);
#pragma unroll
    for (int q = 0; q < R; ++q) out[q * p.ns] = v[b * R + q];
  });
}

// A whole pass in place (TW: not the first), ending with a barrier; the caller has a barrier before it.
template <int EPT, int T, bool TW>
__device__ __forceinline__ void gen_pass(float2* buf, int stride, const float2* tw, const GPass& p, int rb) {
  gen_radix<EPT >= 16 ? 16 : 12>(p.r, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    const int tid = gen_tid();
    float2 v[R * gen_per_thread(R, EPT)];
    gen_read<R, EPT, T>(tid, v, buf, stride, p, rb);
    gen_compute<R, EPT, T, TW>(tid, v, tw, p, rb);
    __syncthreads();
    gen_write<R, EPT, T>(tid, v, buf, stride, p, rb);
  });
  __syncthreads();
}

}  // namespace stem

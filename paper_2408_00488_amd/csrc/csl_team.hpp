// Team transforms and the solver phases built on them (512-thread instances).
//
// A line of n = N - 1 points is transformed by a team of T = N / 8 lanes (T =
// 1 below N = 8), eight points a lane: lane j holds the points m = j + q T, q <
// 8.  Lines of up to 511 points fit a wave, so their teams exchange values
// through LDS with no workgroup barrier (1023 points: two waves and a
// barrier).  A pass through registers is a radix-8 (the first: radix-16)
// Stockham stage, so a line of 511 points meets LDS between three stages instead of
// five, and the waves of a workgroup run independently: the loads and stores
// of one run under the transforms of the others.  (With the workgroup-wide
// radix-4 transform in its place every chunk waited at ten barriers.)
//
//   FP32: the odd extension, an FFT of 2N points with 16 values a lane.  Its
//     first stage folds the extension: x_{m+N} = -x_{N-m}.
//   FP64: the first stage's outputs a = 1 .. 7 (mod 16) and their mirror
//     images 16 - a give every X_k but those with k a multiple of 8, through
//     seven FFTs of T points with half-integer frequencies.  The multiples of
//     8 are the DST-I of T - 1 points x' of the folded line, taken as an eighth
//     FFT of T points of the combined line
//       y_j = sin(pi j / T) (x'_j + x'_{T-j}) + (x'_j - x'_{T-j}) / 2:
//     S_{2m} = i (Y_m - Y_{T-m}) / 2 and the running sum S_{2m+1} = S_{2m-1} +
//     (Y_m + Y_{T-m}) / 2, S_1 = Y_0 / 2.  So a lane holds 8 values where the
//     whole extension takes 16.  The running sum's rounding grows with the
//     square root of its length: with the whole line combined P^{-1} was off by
//     1.9e-14 at 1023^2; over T / 2 <= 64 terms of an eighth of the outputs,
//     closed by S_{T-1} = -Y_{T/2} / 2, and with the inverse factor rounded down
//     (team_cf) it is 5.8e-16 at 1023 x 15 (odd extension 8.5e-16), 5.3e-16 at
//     255^2 (9.6e-16).  255^3: 73.4 -> 72.5 ms, 1023^2: 1.60 -> 1.58 ms.  In FP32 the sum would show (1.5e-7 against 1.1e-7 a transform
//     of 511 points), for no time gained, so FP32 takes the extension.
//
// The vectors Tq, Tv and T are stored column by column: element (row, c) at
// c ld + row, ld = S.ld an odd multiple of 8 (so that the 128-byte runs of
// eight rows that a row phase writes are whole cache lines, and the runs of
// neighbouring columns fall on different memory channels).
#pragma once
#include "csl_device.hpp"

namespace csl {
namespace CSL_KNS {

// LDS of a workgroup: line buffers (line g at g LS elements, LS = N + 1 FP64,
// 2N + 2 FP32: the odd part spreads the transposed accesses of the row phases
// over the banks), then the twiddles exp(-2 pi i k / 2048), k < 512, in FP64
// and in FP32 (a quarter turn; the rest by symmetry), staged once per kernel
// (the team's own table loads would each miss the L2 that the phase's acquire
// has just emptied).
constexpr int kTeamTwLg = 11;
template <typename R> __device__ __forceinline__ const Cx<R> *team_tw(const char *smem) {
  return reinterpret_cast<const Cx<R> *>(smem + kTeamBufBytes + (sizeof(R) == 8 ? 0 : 8192));
}

template <bool F32>
__device__ __forceinline__ void team_stage_twiddles(char *smem) {
  Cx<double> *t64 = const_cast<Cx<double> *>(team_tw<double>(smem));
  Cx<float> *t32 = const_cast<Cx<float> *>(team_tw<float>(smem));
  for (int i = threadIdx.x; i < 512; i += NT) {
    t64[i] = ldg(gbl(twiddles<double>()) + i);
    if (F32) t32[i] = ldg(gbl(twiddles<float>()) + i);
  }
  __syncthreads();
}

// exp(-2 pi i idx / 2048) for idx below a quarter turn / half a turn
template <typename R>
__device__ __forceinline__ Cx<R> tw_q(const char *smem, int idx) {
  return team_tw<R>(smem)[idx];
}
template <typename R>
__device__ __forceinline__ Cx<R> tw_h(const char *smem, int idx) {
  constexpr int Q = 1 << (kTeamTwLg - 2);
  const Cx<R> w = tw_q<R>(smem, idx & (Q - 1));
  return idx < Q ? w : Cx<R>{w.y, -w.x};
}
// Position of element p of a line in its buffer: an XOR within aligned runs
// of 128 bytes, so that the strided Stockham writes (8 or 16 elements between
// lanes) fall on all banks; consecutive elements stay within their run.
template <typename R> __device__ __forceinline__ int swz(int p);
template <> __device__ __forceinline__ int swz<double>(int p) { return p ^ ((p >> 3) & 7); }
template <> __device__ __forceinline__ int swz<float>(int p) { return p ^ ((p >> 4) & 15); }

// Points of a lane whose operands are in flight together: the stencil of K_X,
// the recurrence of the first strided pass, the paired update of K_Z (two waves
// a SIMD, 256 registers each).
constexpr int UX = 4;
constexpr int UY = 8;
constexpr int UZ = 4;

struct Team {
  int n, N, lgT, T;
  int g, j;       // team of this thread, lane within it
  int LS;         // line stride in the buffer
};

// Hide the lane index from the optimiser, so that addresses are formed where
// they are used and not carried in registers across the steps of a round
// (carried, they spill: 1072 bytes a lane in the 2-D instance).
__device__ __forceinline__ void team_fresh(Team &t) { asm volatile("" : "+v"(t.j)); }

// Keep the scheduler from interleaving what stands before with what follows
// (all of a round's divisions or butterflies at once exceed the registers).
__device__ __forceinline__ void team_fence() { __builtin_amdgcn_sched_barrier(0); }

// Order a team's LDS accesses around an exchange.
__device__ __forceinline__ void team_sync(Team &t) {
  if (t.T > 64) __syncthreads();
  else wave_lds_sync();
  team_fresh(t);
}

template <typename R>
__device__ __forceinline__ Team make_team(int n) {
  Team t;
  t.n = n;
  t.N = n + 1;
  const int lgN = ilog2i(t.N);
  t.lgT = lgN > 3 ? lgN - 3 : 0;
  t.T = 1 << t.lgT;
  t.g = threadIdx.x >> t.lgT;
  t.j = threadIdx.x & (t.T - 1);
  const int Nb = t.N > 8 ? t.N : 8;   // a lane's eight points, also where the line has three
  t.LS = sizeof(R) == 8 ? Nb + 1 : 2 * Nb + 2;
  return t;
}

// Some team of this wave works on one of the G lines of a round (teams of
// more than a wave meet at workgroup barriers, so every wave takes part).
__device__ __forceinline__ bool wave_on(const Team &t, int G) {
  return t.T > 64 || (((int)threadIdx.x & ~63) >> t.lgT) < G;
}

template <typename R>
__device__ __forceinline__ Cx<R> mul_mi(Cx<R> a) { return Cx<R>{a.y, -a.x}; }   // -i a

template <typename R>
__device__ __forceinline__ void dft4(Cx<R> &x0, Cx<R> &x1, Cx<R> &x2, Cx<R> &x3) {
  const Cx<R> t0 = cadd(x0, x2), t1 = csub(x0, x2);
  const Cx<R> t2 = cadd(x1, x3), t3 = mul_mi(csub(x1, x3));
  x0 = cadd(t0, t2);
  x1 = cadd(t1, t3);
  x2 = csub(t0, t2);
  x3 = csub(t1, t3);
}

// x[p] -> X[p], natural order on both sides
template <typename R>
__device__ __forceinline__ void dft8(Cx<R> (&x)[8]) {
  constexpr R h = (R)0.70710678118654752440;
  Cx<R> e0 = x[0], e1 = x[2], e2 = x[4], e3 = x[6];
  Cx<R> o0 = x[1], o1 = x[3], o2 = x[5], o3 = x[7];
  dft4(e0, e1, e2, e3);
  dft4(o0, o1, o2, o3);
  o1 = Cx<R>{h * (o1.x + o1.y), h * (o1.y - o1.x)};
  o2 = mul_mi(o2);
  o3 = Cx<R>{h * (o3.y - o3.x), -h * (o3.x + o3.y)};
  x[0] = cadd(e0, o0);
  x[4] = csub(e0, o0);
  x[1] = cadd(e1, o1);
  x[5] = csub(e1, o1);
  x[2] = cadd(e2, o2);
  x[6] = csub(e2, o2);
  x[3] = cadd(e3, o3);
  x[7] = csub(e3, o3);
}

// One Stockham stage of radix RAD on the lane's E values a[q] = element j + q
// T of E T points: E / RAD butterflies b = j + s T of the elements b + p F / RAD
// (q = s + p E / RAD), k = b mod Ns, with the twiddles exp(-2 pi i k' p / (RAD
// Ns)).  k' = k for an FFT of the extended line (E = 16); k' = k - (k mod 8) / 2
// after the folded first stage (E = 8), whose residues stand for half-integer
// frequencies.
template <typename R, int E, int RAD>
__device__ __forceinline__ void team_stage(Cx<R> (&a)[E], const char *smem, int j, int T, int lgNs) {
  constexpr int S = E / RAD;
  constexpr int lgR = RAD == 8 ? 3 : (RAD == 4 ? 2 : 1);
#pragma unroll
  for (int s = 0; s < S; ++s) {
    team_fence();
    const int k = (j + s * T) & ((1 << lgNs) - 1);
    const int i1 = E == 8 ? (2 * k - (k & 7)) << (kTeamTwLg - 1 - lgR - lgNs) : k << (kTeamTwLg - lgR - lgNs);
    if constexpr (RAD == 8) {
      Cx<R> x[8];
      const Cx<R> w1 = tw_q<R>(smem, i1), w2 = tw_q<R>(smem, 2 * i1), w4 = tw_h<R>(smem, 4 * i1);
      const Cx<R> w3 = cmul(w1, w2);
      x[0] = a[s];
      x[1] = cmul(a[s + S], w1);
      x[2] = cmul(a[s + 2 * S], w2);
      x[3] = cmul(a[s + 3 * S], w3);
      x[4] = cmul(a[s + 4 * S], w4);
      x[5] = cmul(a[s + 5 * S], cmul(w1, w4));
      x[6] = cmul(a[s + 6 * S], cmul(w2, w4));
      x[7] = cmul(a[s + 7 * S], cmul(w3, w4));
      dft8(x);
#pragma unroll
      for (int p = 0; p < 8; ++p) a[s + p * S] = x[p];
    } else if constexpr (RAD == 4) {
      const Cx<R> w1 = tw_q<R>(smem, i1), w2 = tw_h<R>(smem, 2 * i1);
      a[s + S] = cmul(a[s + S], w1);
      a[s + 2 * S] = cmul(a[s + 2 * S], w2);
      a[s + 3 * S] = cmul(a[s + 3 * S], cmul(w1, w2));
      dft4(a[s], a[s + S], a[s + 2 * S], a[s + 3 * S]);
    } else {
      const Cx<R> y = cmul(a[s + S], tw_h<R>(smem, i1));
      a[s + S] = csub(a[s], y);
      a[s] = cadd(a[s], y);
    }
  }
}

// The stages after the first (whose output p of lane j is element E j + p): on
// return a[q] = output j + q T.  lb: the line's buffer (E T elements).
// Positions are formed by exclusive or: the lengths and strides are powers of
// two, so the bits of the lane's part and of the (uniform) part of the value
// never meet.
template <typename R, int E>
__device__ __forceinline__ void team_fft_rest(Cx<R> (&a)[E], Cx<R> *lb, const char *smem, Team &t) {
  if (t.T == 1) return;
  const int T = t.T;
  team_sync(t);
  const int w0 = swz<R>(E * t.j);
#pragma unroll
  for (int p = 0; p < E; ++p) lb[w0 ^ p] = a[p];
  team_sync(t);
  const int r0 = swz<R>(t.j);
#pragma unroll
  for (int q = 0; q < E; ++q) a[q] = lb[r0 ^ swz<R>(q * T)];
  int lgNs = E == 8 ? 3 : 4, rem = t.lgT;
  for (; rem > 3; rem -= 3, lgNs += 3) {
    team_stage<R, E, 8>(a, smem, t.j, T, lgNs);
    team_sync(t);
    constexpr int S = E / 8;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int b = t.j + s * T, k = b & ((1 << lgNs) - 1);
      const int w1 = swz<R>(((b - k) << 3) + k);
#pragma unroll
      for (int p = 0; p < 8; ++p) lb[w1 ^ swz<R>(p << lgNs)] = a[s + p * S];
    }
    team_sync(t);
    const int r1 = swz<R>(t.j);
#pragma unroll
    for (int q = 0; q < E; ++q) a[q] = lb[r1 ^ swz<R>(q * T)];
  }
  if (rem == 3) team_stage<R, E, 8>(a, smem, t.j, T, lgNs);
  else if (rem == 2) team_stage<R, E, 4>(a, smem, t.j, T, lgNs);
  else team_stage<R, E, 2>(a, smem, t.j, T, lgNs);
}

// n = 3: the three outputs of a line held by one lane, (x_1, x_2, x_3) ->
// sqrt(1/2) sum_m x_m sin(pi m k / 4)
template <typename R>
__device__ __forceinline__ void dst3(const Cx<R> *lb, Cx<R> (&o)[8]) {
  constexpr R h = (R)0.70710678118654752440;
  const Cx<R> x1 = lb[swz<R>(1)], x2 = lb[swz<R>(2)], x3 = lb[swz<R>(3)];
  const Cx<R> s = {(R)0.5 * (x1.x + x3.x), (R)0.5 * (x1.y + x3.y)};
  const Cx<R> d = {h * x2.x, h * x2.y};
  o[0] = Cx<R>{0, 0};
  o[1] = cadd(s, d);
  o[2] = Cx<R>{h * (x1.x - x3.x), h * (x1.y - x3.y)};
  o[3] = csub(s, d);
#pragma unroll
  for (int q = 4; q < 8; ++q) o[q] = Cx<R>{0, 0};
}

// n = 7 in FP64, held by one lane: the sums u_m = x_m + x_{8-m} give the odd
// outputs, the differences v_m the even ones, X_k = 1/2 sum_m x_m sin(pi m k / 8)
__device__ __forceinline__ void dst7(const Cx<double> *lb, Cx<double> (&o)[8]) {
  constexpr double h = 0.70710678118654752440, c = 0.92387953251128675613, s = 0.38268343236508977173;
  Cx<double> x[8];
#pragma unroll
  for (int m = 1; m < 8; ++m) x[m] = lb[m];   // swz(m) = m below 8
  auto part = [&](auto get, auto put) {
    const double u1 = get(x[1]) + get(x[7]), u2 = get(x[2]) + get(x[6]), u3 = get(x[3]) + get(x[5]);
    const double v1 = get(x[1]) - get(x[7]), v2 = get(x[2]) - get(x[6]), v3 = get(x[3]) - get(x[5]);
    const double u4 = get(x[4]), hu = h * u2, hv = h * (v1 + v3);
    const double p = s * u1 + c * u3, q = c * u1 - s * u3;
    put(o[1], 0.5 * ((p + hu) + u4));
    put(o[7], 0.5 * ((p - hu) - u4));
    put(o[3], 0.5 * ((q + hu) - u4));
    put(o[5], 0.5 * ((q - hu) + u4));
    put(o[2], 0.5 * (hv + v2));
    put(o[6], 0.5 * (hv - v2));
    put(o[4], 0.5 * (v1 - v3));
  };
  part([](const Cx<double> &a) { return a.x; }, [](Cx<double> &a, double b) { a.x = b; });
  part([](const Cx<double> &a) { return a.y; }, [](Cx<double> &a, double b) { a.y = b; });
  o[0] = Cx<double>{0, 0};
}

// First stage, radix 16 on x_m and x_{m+N} = -x_{N-m} (m = j + q T): e[r] =
// output 2r, from x_m - x_{N-m}; d[r] = output 2r + 1, from (x_m + x_{N-m})
// exp(-2 pi i q / 16).  The line starts at swz(m) in its buffer.
__device__ __forceinline__ void team_first(const Cx<double> *lb, const Team &t, Cx<double> (&e)[8],
                                           Cx<double> (&d)[8]) {
  typedef double R;
  constexpr R c1 = (R)0.92387953251128675613, s1 = (R)0.38268343236508977173;
  constexpr R h = (R)0.70710678118654752440;
  const int T = t.T;
  const bool first = t.j == 0;
  const int r0 = swz<R>(t.j), m0 = swz<R>((T - t.j) & (T - 1));
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    // N - m = (T - j) + (7 - q) T (lane 0: (8 - q) T)
    Cx<R> x = lb[r0 ^ swz<R>(q * T)];
    Cx<R> y = lb[m0 ^ (first ? swz<R>(((8 - q) & 7) * T) : swz<R>((7 - q) * T))];
    if (q == 0 && first) x = y = Cx<R>{0, 0};
    e[q] = csub(x, y);
    d[q] = cadd(x, y);
  }
  d[1] = cmul(d[1], Cx<R>{c1, -s1});
  d[2] = Cx<R>{h * (d[2].x + d[2].y), h * (d[2].y - d[2].x)};
  d[3] = cmul(d[3], Cx<R>{s1, -c1});
  d[4] = mul_mi(d[4]);
  d[5] = cmul(d[5], Cx<R>{-s1, -c1});
  d[6] = Cx<R>{h * (d[6].y - d[6].x), -h * (d[6].x + d[6].y)};
  d[7] = cmul(d[7], Cx<R>{-c1, -s1});
  team_fence();
  dft8(e);
  team_fence();
  dft8(d);
  team_fence();
}

// 1 / sqrt(2 N), N = 8 T > 8.  Where it is not a power of two an inverse transform
// takes sqrt(1/2) rounded down: the factors of a transform and its inverse are
// the same for every value, and with both rounded up their product would be off
// by 1.4e-16 (so: by -2e-17).
__device__ __forceinline__ double team_cf(const Team &t, bool inverse) {
  const int lg = t.lgT + 4;
  const double h = inverse ? 0.70710678118654746 : 0.70710678118654757;
  return ldexp((lg & 1) ? h : 1.0, -(lg >> 1));
}

// Orthonormal DST-I of the team's line, held in its buffer (x_m at swz(m), m =
// 1 .. N - 1): o[q] = X_{j + q T} (o[0] of lane 0 is no output).  Starts by
// ordering the team's writes of the line; the buffer may be written again by
// the team once its outputs are used.
__device__ __forceinline__ void team_dst(Cx<float> *lb, const char *smem, Team &t, Cx<float> (&o)[8],
                                         bool) {
  typedef float R;
  team_sync(t);
  if (t.N == 4) {
    dst3<R>(lb, o);
    return;
  }
  Cx<R> a[16];
  {
    // first stage, radix 16 on x_m and x_{m+N} = -x_{N-m}: outputs 2r from
    // s_q = x_m - x_{N-m}, 2r + 1 from d_q = (x_m + x_{N-m}) exp(-2 pi i q / 16)
    constexpr R c1 = (R)0.92387953251128675613, s1 = (R)0.38268343236508977173;
    constexpr R h = (R)0.70710678118654752440;
    Cx<R> s[8], d[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int m = t.j + q * t.T;
      Cx<R> x = lb[swz<R>(m)], y = lb[swz<R>(t.N - m)];
      if (q == 0 && m == 0) x = y = Cx<R>{0, 0};
      s[q] = csub(x, y);
      d[q] = cadd(x, y);
    }
    d[1] = cmul(d[1], Cx<R>{c1, -s1});
    d[2] = Cx<R>{h * (d[2].x + d[2].y), h * (d[2].y - d[2].x)};
    d[3] = cmul(d[3], Cx<R>{s1, -c1});
    d[4] = mul_mi(d[4]);
    d[5] = cmul(d[5], Cx<R>{-s1, -c1});
    d[6] = Cx<R>{h * (d[6].y - d[6].x), -h * (d[6].x + d[6].y)};
    d[7] = cmul(d[7], Cx<R>{-c1, -s1});
    team_fence();
    dft8(s);
    team_fence();
    dft8(d);
    team_fence();
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      a[2 * r] = s[r];
      a[2 * r + 1] = d[r];
    }
  }
  team_fft_rest<R, 16>(a, lb, smem, t);
  const R cf = (R)1 / sqrt((R)(2 * t.N));
#pragma unroll
  for (int q = 0; q < 8; ++q) o[q] = dst_out(a[q], cf);
}

// FP64: the outputs are left in the buffer (X_k at swz(k)).
__device__ __forceinline__ void team_dst_lds(Cx<double> *lb, const char *smem, Team &t, bool inverse) {
  typedef double R;
  team_sync(t);
  if (t.N <= 8) {
    Cx<R> o[8];
    if (t.N == 4) dst3<R>(lb, o);
    else dst7(lb, o);
    team_sync(t);
#pragma unroll
    for (int q = 1; q < 8; ++q) lb[q] = o[q];
    return;
  }
  const int T = t.T;
  const R cf = team_cf(t, inverse);
  Cx<R> a[8];
  {
    Cx<R> e[8], d[8];
    team_first(lb, t, e, d);
    const R sn = -tw_h<R>(smem, t.j << (kTeamTwLg - 1 - t.lgT)).y;
    a[0] = Cx<R>{sn * e[4].x + 0.5 * e[0].x, sn * e[4].y + 0.5 * e[0].y};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (r) a[2 * r] = e[r];
      a[2 * r + 1] = d[r];
    }
  }
  team_fft_rest<R, 8>(a, lb, smem, t);
  team_sync(t);
#pragma unroll
  for (int q = 0; q < 8; ++q) a[q] = dst_out(a[q], q < 4 ? cf : -cf);
  // output K = j + q T belongs to k = 16 (K / 8) + K mod 8, above N to 2N - k;
  // those with K mod 8 = 0 wait at K
  if (T >= 8) {
    const bool z = (t.j & 7) == 0;
    const int f = ((t.j >> 3) << 4) | (t.j & 7);
    const int p0 = swz<R>(z ? t.j : f), p1 = swz<R>(z ? t.j : 2 * T - f);
#pragma unroll
    for (int q = 0; q < 8; ++q)
      lb[(q < 4 ? p0 : p1) ^ (z ? swz<R>(q * T) : swz<R>((q < 4 ? q : 7 - q) * 2 * T))] = a[q];
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int K = t.j + q * T, k = 2 * K - (K & 7);
      lb[swz<R>((K & 7) == 0 ? K : (k < t.N ? k : 2 * t.N - k))] = a[q];
    }
  }
  // residue 0: X_{16 m} and X_{16 m + 8} (a running sum), m < T / 2, the real
  // parts' sources in the lower half of the lanes, the imaginary in the upper;
  // the last sum is Y_{T/2} too, and what the rounding leaves between the two is
  // spread over the sums
  team_sync(t);
  const int H = T >> 1, m = t.j & (H - 1), c = t.j >= H;
  R *lr = reinterpret_cast<R *>(lb);
  const R y = lr[2 * swz<R>(8 * m) + c];
  R z = lr[2 * swz<R>((8 * (T - m)) & (8 * T - 1)) + c];
  const R e = lr[2 * swz<R>(4 * T) + c];
  if (m == 0) z = 0;
  R run = c ? y - z : z - y;
  for (int d = 1; d < H; d <<= 1) {
    const R u = __shfl_up(run, (unsigned)d, H);
    if (m >= d) run += u;
  }
  const R last = __shfl(run, H - 1, H);
  run += ((c ? e : -e) - last) * ((m + 0.5) / H);
  team_sync(t);
  if (m) lr[2 * swz<R>(16 * m) + c] = y + z;
  lr[2 * swz<R>(16 * m + 8) + 1 - c] = run;
}

__device__ __forceinline__ void team_dst(Cx<double> *lb, const char *smem, Team &t, Cx<double> (&o)[8],
                                         bool inverse) {
  typedef double R;
  team_dst_lds(lb, smem, t, inverse);
  team_sync(t);
  const int r0 = swz<R>(t.j);
#pragma unroll
  for (int q = 0; q < 8; ++q) o[q] = lb[t.N == 4 ? swz<R>(q & 3) : r0 ^ swz<R>(q * t.T)];
}

// Index of the point m = j + q T of a team's line, kept inside the line (lane 0
// has no point at q = 0, a line of three points none past q = 3), so that the
// loads of a round need no branches; what they bring in there is not used.
__device__ __forceinline__ int team_idx(const Team &t, int q) {
  const int i = t.j + q * t.T - 1;
  if (q == 0) return max(i, 0);
  return q < 4 ? i : min(i, t.n - 1);
}
// The point exists (q < 4: in every line).
__device__ __forceinline__ bool team_pt0(const Team &t, int q) { return q > 0 || t.j > 0; }

// Stencil operands of a point without branches: neighbours outside the grid
// are replaced by the point itself on loading and by zero on use.
template <int D>
__device__ __forceinline__ StencilIn<D> stencil_load_flat(const SysDesc &S,
                                                          const CSL_G double2 *__restrict__ u, int p,
                                                          const int (&idx)[3]) {
  StencilIn<D> in;
  const CSL_G double *__restrict__ A = gbl(S.a);
  in.c = ldg(u + p);
  in.ap = A[p];
  in.inb = 0u;
  in.ina = 0u;
#pragma unroll
  for (int ax = 0; ax < D; ++ax) {
    const int st = S.st[ax];
    const bool lo = idx[ax] > 0, hi = idx[ax] < S.n[ax] - 1;
    in.inb |= (lo ? 1u : 0u) << ax;
    in.ina |= (hi ? 1u : 0u) << ax;
    const int pb = lo ? p - st : p, pa = hi ? p + st : p;
    in.b[ax] = ldg(u + pb);
    in.a[ax] = ldg(u + pa);
    in.ab[ax] = A[pb];
    in.aa[ax] = A[pa];
  }
  return in;
}

// n / d for a face coefficient, n = 2 a b and d = a + b of positive samples: the
// hardware's reciprocal refined to the last bit or two, the quotient from it and
// one correction by its residual (Markstein's division).  The result is the
// division's (no difference in 4e6 pairs between 1e-150 and 1e150; one unit in
// the last place where n is subnormal).  The operands are not scaled, which a
// face does not need: where d is below the normal range n is 0.  With the
// compiler's division a small solve takes 5% longer (63^2 FP64, 30 steps: 0.90
// ms, 0.86 here) and the 3-D instance spills.  One reciprocal 1 / (s1 s2) for both
// faces of an axis (0.87 ms) rounds more (rms error of a face 1.2e-16 against
// 0.9e-16) and overflows where samples differ by 1e200.
__device__ __forceinline__ double face_div(double n, double d) {
  d = fmax(d, 2.2250738585072014e-308);
  double r = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, r, 1.0);
  r = fma(r, fma(e, e, e), r);
  const double q = n * r;
  return fma(fma(-q, d, n), r, q);
}

// The operator of stencil_apply; the products are fused into the sum one by one
// (a rounding each, whatever the compiler contracts), as in the recurrence of
// the first strided pass.
template <int D>
__device__ __forceinline__ double2 stencil_apply_flat(const SysDesc &S, const StencilIn<D> &in) {
  double rx = 0.0, ry = 0.0;
#pragma unroll
  for (int ax = 0; ax < D; ++ax) {
    team_fence();
    const double h2 = S.h2[ax];
    const bool lo = (in.inb >> ax) & 1u, hi = (in.ina >> ax) & 1u;
    const double hb = face_div(2.0 * in.ab[ax] * in.ap, in.ab[ax] + in.ap);
    const double ha = face_div(2.0 * in.ap * in.aa[ax], in.ap + in.aa[ax]);
    const double fb = (lo ? hb : in.ap) * h2, fa = (hi ? ha : in.ap) * h2;
    rx = fma(fa, in.c.x - (hi ? in.a[ax].x : 0.0), fma(fb, in.c.x - (lo ? in.b[ax].x : 0.0), rx));
    ry = fma(fa, in.c.y - (hi ? in.a[ax].y : 0.0), fma(fb, in.c.y - (lo ? in.b[ax].y : 0.0), ry));
  }
  return make_double2(rx, ry);
}

// ---------------------------------------------------------------------------
// K_X: rows of the contiguous axis, FP64 (see tile_X): a round is S.lpt_x rows,
// one per team.  Every team forms the stencil values of its row and
// transforms them; then the workgroup stores the round's rows, rows fastest
// (the columns of Tq are contiguous).
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void tile_TX(const SysDesc &S, const IOPtr &io, int iter, int tile, char *smem,
                                        double *red) {
  Team t = make_team<double>(S.n[D - 1]);
  const int G = S.lpt_x, lgG = ilog2i(G);
  Cx<double> *buf = reinterpret_cast<Cx<double> *>(smem);
  const bool on = wave_on(t, G);
  Cx<double> *lb = buf + t.g * t.LS;
  const int r0 = tile * S.cpt[K_X] * G, r1 = min(S.rows, (tile + 1) * S.cpt[K_X] * G);
  const int ld = S.ld, n = t.n;
  const double al = S.alpha, be = S.beta;
  const CSL_G double2 *__restrict__ zj = gbl(S.Z[iter & 1]);
  const CSL_G double2 *__restrict__ f = gbl(io.f);
  CSL_G double2 *__restrict__ X = gbl(io.x);
  CSL_G double2 *__restrict__ out = gbl(iter == 0 ? S.Tv[1] : S.Tq);
  double acc = 0.0;
  for (int rb = r0; rb < r1; rb += G) {
    const bool act = t.g < G && rb + t.g < r1;
    const int row = min(rb + t.g, r1 - 1);
    team_fresh(t);
    if (on) {
      if (iter == 0) {
        double2 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = ldg(f + (row * n + team_idx(t, q)));
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          lb[swz<double>(t.j + q * t.T)] = Cx<double>{v[q].x, v[q].y};
          if (act && team_pt0(t, q) && (q < 4 || t.N > 4)) {
            acc += v[q].x * v[q].x + v[q].y * v[q].y;
            st_nt(X + (row * n + team_idx(t, q)), 0.0, 0.0);
          }
        }
      } else {
#pragma unroll
        for (int q0 = 0; q0 < 8; q0 += UX) {
          StencilIn<D> in[UX];
          team_fence();
#pragma unroll
          for (int u = 0; u < UX; ++u) {
            const int i = team_idx(t, q0 + u);
            int idx[3];
            row_index<D>(S, row, i, idx);
            in[u] = stencil_load_flat<D>(S, zj, row * n + i, idx);
          }
#pragma unroll
          for (int u = 0; u < UX; ++u) {
            team_fence();
            const int q = q0 + u;
            const double2 kz = stencil_apply_flat<D>(S, in[u]);
            const double2 zz = in[u].c;
            const double qx = kz.x + al * zz.x + be * zz.y;
            const double qy = -(kz.y + al * zz.y - be * zz.x);
            const double d = zz.x * qx + zz.y * qy;
            acc += (act && team_pt0(t, q) && (q < 4 || t.N > 4)) ? d : 0.0;
            lb[swz<double>(t.j + q * t.T)] = Cx<double>{qx, qy};
          }
        }
      }
      team_dst_lds(lb, smem, t, false);
    }
    __syncthreads();
    const int R = min(G, r1 - rb);
    for (int e = threadIdx.x; e < (n << lgG); e += NT) {
      const int rr = e & (G - 1), k = e >> lgG;
      if (rr < R) {
        const Cx<double> v = buf[rr * t.LS + swz<double>(k + 1)];
        st_nt(out + (k * ld + rb + rr), v.x, v.y);
      }
    }
    __syncthreads();
  }
  const double s = wg_sum(acc, red);
  if (threadIdx.x == 0) red[NT / 64] = s;
}

// Factor of P^{-1} for the mode with the eigenvalue sum lam.
template <typename R>
__device__ __forceinline__ R mode_factor(R lam, R ab, R al, R be) {
  const R sh = ab * lam + al;
  return (R)1 / sqrt(sh * sh + be * be);
}

template <typename R> __device__ __forceinline__ const CSL_G R *mode_mu(const SysDesc &S, int ax);
template <> __device__ __forceinline__ const CSL_G double *mode_mu<double>(const SysDesc &S, int ax) {
  return gbl(S.mu[ax]);
}
template <> __device__ __forceinline__ const CSL_G float *mode_mu<float>(const SysDesc &S, int ax) {
  return gbl(S.mu_f[ax]);
}

// Scale the transformed line by its modes' factors (m12: the sum of the other
// axes' eigenvalues) and put it back in the buffer; returns the lane's share
// of sum_k s_k |U_k|^2 (0 unless act).
template <typename R>
__device__ __forceinline__ void team_mu0(const SysDesc &S, const Team &t, R (&mu)[8]) {
  const CSL_G R *mu0 = mode_mu<R>(S, 0);
#pragma unroll
  for (int q = 0; q < 8; ++q) mu[q] = mu0[team_idx(t, q)];
}
template <typename R, class Lam>
__device__ __forceinline__ double team_scale(const SysDesc &S, Cx<R> *lb, Team &t, const Cx<R> (&o)[8],
                                             const R (&mu)[8], bool act, Lam &&lam) {
  const R ab = sizeof(R) == 8 ? (R)S.abar : (R)S.abar_f;
  const R al = sizeof(R) == 8 ? (R)S.alpha : (R)S.alpha_f;
  const R be = sizeof(R) == 8 ? (R)S.beta : (R)S.beta_f;
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    team_fence();
    const R s = mode_factor<R>(lam(mu[q]), ab, al, be);
    const double d = (double)s * ((double)o[q].x * (double)o[q].x + (double)o[q].y * (double)o[q].y);
    acc += (act && team_pt0(t, q) && (q < 4 || t.N > 4)) ? d : 0.0;
    lb[swz<R>(t.j + q * t.T)] = Cx<R>{o[q].x * s, o[q].y * s};
  }
  return acc;
}

// ---------------------------------------------------------------------------
// Strided passes, preconditioner precision R (see tile_Y).  Lines along axis
// D - 2 are contiguous in the column order, so a team reads and writes its
// line itself: 2-D K_Y (lines = columns), 3-D K_Y1 and K_Y1I (line c n0 + i0).
// No workgroup barrier for lines of at most 511 points.
// ---------------------------------------------------------------------------
template <typename R, int D>
__device__ __forceinline__ void tile_TY(const SysDesc &S, const Ctl *C, int kind, int iter, int tile, char *smem,
                                        double *red) {
  constexpr int ax = D - 2;
  Team t = make_team<R>(S.n[ax]);
  const int G = S.lpt_s[ax];
  const bool on = wave_on(t, G);
  Cx<R> *lb = reinterpret_cast<Cx<R> *>(smem) + t.g * t.LS;
  const int nlines = D == 2 ? S.n[1] : S.n[2] * S.n[0];
  const int l0 = tile * S.cpt[kind] * G, l1 = min(nlines, (tile + 1) * S.cpt[kind] * G);
  const int ld = S.ld, n = t.n;
  CSL_G Cx<R> *T = gbl(reinterpret_cast<Cx<R> *>(S.T));
  const bool first = kind == K_Y1 || D == 2;
  CSL_G double2 *vout = gbl(S.Tv[(iter + 1) & 1]);   // holds Tv_{j-1}
  const CSL_G double2 *vj = gbl(S.Tv[iter & 1]);
  // iteration 0: the line is Tv_1 itself; iteration 1 has no Tv_0 (its
  // factor is 0, the operand any finite vector)
  const CSL_G double2 *tq = iter == 0 ? gbl(S.Tv[1]) : gbl(S.Tq);
  const CSL_G double2 *vm = iter >= 2 ? vout : tq;
  double cd = 0.0, cg = 0.0;
  if (first && iter > 0) {
    const double g = ld_ctl(&C->gamma), go = ld_ctl(&C->gamma_old);
    cd = ld_ctl(&C->delta) / g;
    cg = iter >= 2 ? g / go : 0.0;
  }
  double gacc = 0.0;
  for (int lbs = l0; lbs < l1; lbs += G) {
    const bool act = t.g < G && lbs + t.g < l1;
    const int line = min(lbs + t.g, l1 - 1);
    team_fresh(t);
    if (on) {
      const int c = D == 2 ? line : line / S.n[0];
      const int base = D == 2 ? line * ld : c * ld + (line - c * S.n[0]) * n;
      R mu[8], m1 = 0;
      if constexpr (D == 2) {
        team_mu0<R>(S, t, mu);   // ahead of the transform that it follows
        m1 = mode_mu<R>(S, 1)[c];
      }
      if (!first) {
        Cx<R> v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = ldg(T + (base + team_idx(t, q)));
#pragma unroll
        for (int q = 0; q < 8; ++q) lb[swz<R>(t.j + q * t.T)] = v[q];
      } else if (iter == 0) {
        double2 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = ldg(tq + (base + team_idx(t, q)));
#pragma unroll
        for (int q = 0; q < 8; ++q) lb[swz<R>(t.j + q * t.T)] = Cx<R>{(R)v[q].x, (R)v[q].y};
      } else {
#pragma unroll
        for (int q0 = 0; q0 < 8; q0 += UY) {
          double2 a[UY], b[UY], d[UY];
          team_fence();
#pragma unroll
          for (int u = 0; u < UY; ++u) {
            const int p = base + team_idx(t, q0 + u);
            a[u] = ldg(tq + p);
            b[u] = ldg(vj + p);
            d[u] = ldg(vm + p);
          }
#pragma unroll
          for (int u = 0; u < UY; ++u) {
            a[u].x = fma(-cg, d[u].x, fma(-cd, b[u].x, a[u].x));
            a[u].y = fma(-cg, d[u].y, fma(-cd, b[u].y, a[u].y));
            lb[swz<R>(t.j + (q0 + u) * t.T)] = Cx<R>{(R)a[u].x, (R)a[u].y};
          }
          if (act) {
#pragma unroll
            for (int u = 0; u < UY; ++u)
              if (team_pt0(t, q0 + u) && (q0 + u < 4 || t.N > 4))
                st_nt(vout + (base + team_idx(t, q0 + u)), a[u].x, a[u].y);
          }
        }
      }
      Cx<R> o[8];
      team_dst(lb, smem, t, o, kind == K_Y1I);
      if constexpr (D == 2) {
        team_sync(t);
        gacc += team_scale<R>(S, lb, t, o, mu, act, [&](R m0) { return m0 + m1; });
        team_dst(lb, smem, t, o, true);
      }
      if (act) {
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (team_pt0(t, q) && (q < 4 || t.N > 4)) st_nt(T + (base + team_idx(t, q)), o[q]);
      }
      // the next round's line replaces this one's values
      team_sync(t);
    }
  }
  if (kind == K_Y) {
    const double sg = wg_sum(gacc, red);
    if (threadIdx.x == 0) red[NT / 64] = sg;
  }
}

// 3-D K_Y: lines along axis 0 (stride n1 in the column order): a round is
// lpt_s[0] neighbouring lines i1 of one column c, read and written by the
// workgroup with i1 fastest and transformed by a team each.
template <typename R>
__device__ __forceinline__ void tile_TY0(const SysDesc &S, int tile, char *smem, double *red) {
  Team t = make_team<R>(S.n[0]);
  const int G = S.lpt_s[0], lgG = ilog2i(G);
  Cx<R> *buf = reinterpret_cast<Cx<R> *>(smem);
  const bool on = wave_on(t, G);
  Cx<R> *lb = buf + t.g * t.LS;
  const int n1 = S.n[1], n = t.n;
  const int ngrp = (n1 + G - 1) >> lgG;
  const int c0 = tile * S.cpt[K_Y], c1 = min(S.nchunk[K_Y], (tile + 1) * S.cpt[K_Y]);
  CSL_G Cx<R> *T = gbl(reinterpret_cast<Cx<R> *>(S.T));
  double gacc = 0.0;
  for (int ch = c0; ch < c1; ++ch) {
    const int c = ch / ngrp, i1b = (ch - c * ngrp) << lgG;
    const int L = min(G, n1 - i1b);
    CSL_G Cx<R> *Tc = T + (c * S.ld + i1b);
    constexpr int U = 8;
    for (int e0 = threadIdx.x; e0 < (n << lgG); e0 += NT * U) {
      Cx<R> v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * NT, rr = min(e & (G - 1), L - 1), k = min(e >> lgG, n - 1);
        v[u] = ldg(Tc + (k * n1 + rr));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * NT, rr = e & (G - 1), k = e >> lgG;
        if (k < n) buf[rr * t.LS + swz<R>(k + 1)] = v[u];
      }
    }
    __syncthreads();
    const bool act = t.g < L;
    team_fresh(t);
    if (on) {
      Cx<R> o[8];
      R mu[8];
      team_mu0<R>(S, t, mu);
      const R m1 = mode_mu<R>(S, 1)[min(i1b + t.g, n1 - 1)];
      const R m2 = mode_mu<R>(S, 2)[c];
      team_dst(lb, smem, t, o, false);
      team_sync(t);
      gacc += team_scale<R>(S, lb, t, o, mu, act, [&](R m0) { return (m0 + m1) + m2; });
      team_dst(lb, smem, t, o, true);
      team_sync(t);
#pragma unroll
      for (int q = 0; q < 8; ++q) lb[swz<R>(t.j + q * t.T)] = o[q];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < (n << lgG); e += NT) {
      const int rr = e & (G - 1), k = e >> lgG;
      if (rr < L) st_nt(Tc + (k * n1 + rr), buf[rr * t.LS + swz<R>(k + 1)]);
    }
    __syncthreads();
  }
  const double sg = wg_sum(gacc, red);
  if (threadIdx.x == 0) red[NT / 64] = sg;
}

// ---------------------------------------------------------------------------
// K_Z: rows of the contiguous axis, precision R (see tile_Z): the workgroup
// reads a round's rows of T' (rows fastest) into the line buffers, then every
// team transforms its row and applies the step's update to its points.
// ---------------------------------------------------------------------------
template <typename R, int D>
__device__ __forceinline__ void tile_TZ(const SysDesc &S, const Ctl *C, const IOPtr &io, int iter, int tile,
                                        char *smem) {
  Team t = make_team<R>(S.n[D - 1]);
  const int G = S.lpt_z, lgG = ilog2i(G);
  Cx<R> *buf = reinterpret_cast<Cx<R> *>(smem);
  const bool on = wave_on(t, G);
  Cx<R> *lb = buf + t.g * t.LS;
  const int r0 = tile * S.cpt[K_Z] * G, r1 = min(S.rows, (tile + 1) * S.cpt[K_Z] * G);
  const int ld = S.ld, n = t.n, j = iter;
  const int mode = j == 0 ? ZM_DEFER : ld_ctl(&C->zmode);
  CSL_G double2 *X = gbl(io.x);
  CSL_G double2 *znew = gbl(S.Z[(j + 1) & 1]);
  const CSL_G double2 *zj = gbl(S.Z[j & 1]);
  // ZM_SINGLE: wn holds w_{j-1} and receives w_{j+1}, wo holds w_j;
  // ZM_PAIR: wo holds w_{j-2} and receives w_j, wn holds w_{j-1} and receives
  // w_{j+1} (each entry read before the same lane overwrites it)
  CSL_G double2 *wo = gbl(S.W[j & 1]);
  CSL_G double2 *wn = gbl(S.W[(j + 1) & 1]);
  double e1 = 0, e2 = 0, e3 = 0, ceta = 0, ie1 = 0, e2p = 0, e3p = 0, cetap = 0, ie1p = 0;
  if (mode != ZM_DEFER) {
    e1 = ld_ctl(&C->e1);
    e2 = ld_ctl(&C->e2);
    e3 = ld_ctl(&C->e3);
    ceta = ld_ctl(&C->ceta);
    ie1 = 1.0 / e1;
  }
  if (mode == ZM_FLUSH) {
    // the deferred step m = j - 1 alone: w_j = (zhat_{j-1} - e3 w_{j-2} - e2
    // w_{j-1}) / e1 with step m's coefficients, x += ceta w_j
    const double2 zero = make_double2(0.0, 0.0);
    for (int p = r0 * n + (int)threadIdx.x; p < r1 * n; p += NT) {
      const double2 z = ldg(znew + p);
      const double2 w0 = j > 3 ? ldg(wo + p) : zero;
      const double2 w1 = j > 2 ? ldg(wn + p) : zero;
      const double2 x = j > 2 ? ldg(X + p) : zero;
      const double wx = (z.x - e3 * w0.x - e2 * w1.x) * ie1;
      const double wy = (z.y - e3 * w0.y - e2 * w1.y) * ie1;
      st_nt(wo + p, wx, wy);
      st_nt(X + p, x.x + ceta * wx, x.y - ceta * wy);
    }
    return;
  }
  // operands that do not exist yet (w_0, w_{-1}) get the factor 0 and a finite
  // vector in their place; x_0 = 0 was written at iteration 0
  const CSL_G double2 *wor = wo, *wnr = wn;
  if (mode == ZM_SINGLE) {
    if (j <= 2) {
      e3 = 0.0;
      wnr = zj;
    }
    if (j <= 1) {
      e2 = 0.0;
      wor = zj;
    }
  } else if (mode == ZM_PAIR) {
    e2p = ld_ctl(&C->e2p);
    e3p = ld_ctl(&C->e3p);
    cetap = ld_ctl(&C->cetap);
    ie1p = 1.0 / ld_ctl(&C->e1p);
    if (j <= 3) {
      e3p = 0.0;
      wor = zj;
    }
    if (j <= 2) {
      e2p = 0.0;
      e3 = 0.0;
      wnr = zj;
    }
  }
  const CSL_G Cx<R> *T = gbl(reinterpret_cast<const Cx<R> *>(S.T));
  const double gm = ld_ctl(&C->gamma);
  const bool store_z = (gm != 0.0);
  const double ig = store_z ? 1.0 / gm : 0.0;
  for (int rb = r0; rb < r1; rb += G) {
    const int R_ = min(G, r1 - rb);
    const CSL_G Cx<R> *Tr = T + rb;
    constexpr int U = 8;
    for (int e0 = threadIdx.x; e0 < (n << lgG); e0 += NT * U) {
      Cx<R> v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * NT, rr = min(e & (G - 1), R_ - 1), k = min(e >> lgG, n - 1);
        v[u] = ldg(Tr + (k * ld + rr));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * NT, rr = e & (G - 1), k = e >> lgG;
        if (k < n) buf[rr * t.LS + swz<R>(k + 1)] = v[u];
      }
    }
    __syncthreads();
    const bool act = t.g < G && rb + t.g < r1;
    const int row = min(rb + t.g, r1 - 1);
    team_fresh(t);
    if (on) {
      Cx<R> o[8];
      const int base = row * n;
      double2 zm[UZ], z[UZ], wa[UZ], wb[UZ], x[UZ];
      auto load = [&](int q0) {
#pragma unroll
        for (int u = 0; u < UZ; ++u) {
          const int p = base + team_idx(t, q0 + u);
          zm[u] = ldg(znew + p);   // zhat_{j-1}
          z[u] = ldg(zj + p);
          wa[u] = ldg(wor + p);
          wb[u] = ldg(wnr + p);
          x[u] = ldg(X + p);
        }
      };
      if (mode == ZM_PAIR) load(0);   // ahead of the transform
      team_dst(lb, smem, t, o, true);
      if (mode == ZM_DEFER) {
        if (act) {
#pragma unroll
          for (int q = 0; q < 8; ++q)
            if (team_pt0(t, q) && (q < 4 || t.N > 4))
              st_nt(znew + (base + team_idx(t, q)), (double)o[q].x * ig, (double)o[q].y * ig);
        }
      } else if (mode == ZM_SINGLE) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          team_fence();
          const int p = base + team_idx(t, q);
          const double2 z = ldg(zj + p), w0 = ldg(wnr + p), w1 = ldg(wor + p), x = ldg(X + p);
          const double wx = (z.x - e3 * w0.x - e2 * w1.x) * ie1;
          const double wy = (z.y - e3 * w0.y - e2 * w1.y) * ie1;
          if (act && team_pt0(t, q) && (q < 4 || t.N > 4)) {
            if (store_z) st_nt(znew + p, (double)o[q].x * ig, (double)o[q].y * ig);
            st_nt(wn + p, wx, wy);
            st_nt(X + p, x.x + ceta * wx, x.y - ceta * wy);
          }
        }
      } else {
#pragma unroll
        for (int q0 = 0; q0 < 8; q0 += UZ) {
          team_fence();
          if (q0 > 0) load(q0);
#pragma unroll
          for (int u = 0; u < UZ; ++u) {
            team_fence();
            const int q = q0 + u, p = base + team_idx(t, q);
            const double ax = (zm[u].x - e3p * wa[u].x - e2p * wb[u].x) * ie1p;
            const double ay = (zm[u].y - e3p * wa[u].y - e2p * wb[u].y) * ie1p;
            const double bx = (z[u].x - e3 * wb[u].x - e2 * ax) * ie1;
            const double by = (z[u].y - e3 * wb[u].y - e2 * ay) * ie1;
            const double xx = x[u].x + cetap * ax, xy = x[u].y - cetap * ay;
            if (act && team_pt0(t, q) && (q < 4 || t.N > 4)) {
              if (store_z) st_nt(znew + p, (double)o[q].x * ig, (double)o[q].y * ig);
              st_nt(wo + p, ax, ay);
              st_nt(wn + p, bx, by);
              st_nt(X + p, xx + ceta * bx, xy - ceta * by);
            }
          }
        }
      }
    }
    __syncthreads();
  }
}

}  // namespace CSL_KNS
}  // namespace csl

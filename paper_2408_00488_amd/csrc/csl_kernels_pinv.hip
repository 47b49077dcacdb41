// Stand-alone P^{-1} in FP64 on the team transforms (csl_team.hpp), namespace
// csl::pinv512: the passes of wg256::pinv_pass_kernel (0 rows forward, 1 axis-1
// forward, 2 axis 0 with the mode scaling, 3 axis-1 inverse, 4 rows inverse)
// for grids with the FFT on every axis, T stored column by column.
//
// A pass streams 32 bytes a point (16 read, 16 written) and transforms it once
// (pass 2 twice), so five passes at the card's copy rate are 0.56 ms at 255^3;
// what is left is the latency of a round.  A workgroup walks a run of rounds (a
// line per team), so the twiddles are staged once, and loads the next round's
// values before it transforms the current one.  One workgroup of eight waves a
// CU: two are limited to 128 registers a lane, spill, and are slower (255^3:
// 0.72 against 0.67 ms).  The passes before (a workgroup per 32 KiB chunk, ten
// barriers each) took 1.04 ms at 255^3, 79 us at 1023^2, 48 us at 63^3, 26 us
// at 63^2; these 0.67 ms, 53, 38 and 17 us.
#define CSL_NT 512
#define CSL_KNS pinv512
#define CSL_WAVES_PER_EU 2
#include <algorithm>
#include "csl_team.hpp"
#include "csl_kernels.hpp"

namespace csl {
namespace pinv512 {

typedef CSL_G Cx<double> GC;

template <int D, int PASS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(CSL_WAVES_PER_EU))) void pinv_team_kernel(
    const SysDesc *__restrict__ sys, const double2 *x, double2 *y, int lgG) {
  extern __shared__ __align__(16) char smem[];
  const SysDesc &S = *sys;
  constexpr int ax = (PASS == 0 || PASS == 4) ? D - 1 : (PASS == 2 ? 0 : 1);
  // lines the workgroup reads (writes) itself, lines fastest; the others are
  // read and written by their teams
  constexpr bool strided = PASS == 2 && D == 3;
  constexpr bool wg_read = strided || PASS == 4, wg_write = strided || PASS == 0;
  Team t = make_team<double>(S.n[ax]);
  const int n = t.n, G = 1 << lgG, ld = team_ld(S.rows);
  // rounds of the pass, and lines of a group of rounds (3-D axis 0: the lines i1
  // of one column; else all lines)
  const int lines = strided ? S.n[1] : (ax == D - 1 ? S.rows : (D == 2 ? S.n[1] : S.n[2] * S.n[0]));
  const int per = (lines + G - 1) >> lgG;
  const int rounds = strided ? per * S.n[2] : per;
  const int g0 = (int)((long long)rounds * blockIdx.x / gridDim.x);
  const int g1 = (int)((long long)rounds * (blockIdx.x + 1) / gridDim.x);
  if (g0 >= g1) return;
  team_stage_twiddles<false>(smem);
  Cx<double> *buf = reinterpret_cast<Cx<double> *>(smem);
  const bool on = wave_on(t, G);
  Cx<double> *lb = buf + t.g * t.LS;
  GC *T = gbl(reinterpret_cast<Cx<double> *>(S.T));
  const GC *X = reinterpret_cast<const GC *>(gbl(x));
  GC *Y = reinterpret_cast<GC *>(gbl(y));
  const int stride = strided ? S.n[1] : ld;
  // first element of a round's lines (strided: of column c), its lines
  struct Where {
    int base, l0, L;
  };
  auto where = [&](int r) {
    Where w;
    const int c = strided ? r / per : 0;
    w.l0 = (strided ? r - c * per : r) << lgG;
    w.L = min(G, lines - w.l0);
    w.base = strided ? c * ld + w.l0 : w.l0;
    return w;
  };
  // the team's own line (clamped to the round's)
  auto line_base = [&](const Where &w) {
    const int line = w.l0 + min(t.g, w.L - 1);
    if (ax == D - 1) return line * n;
    if (D == 2) return line * ld;
    const int c = line / S.n[0];
    return c * ld + (line - c * S.n[0]) * n;
  };
  Cx<double> cur[8];   // the round's values, loaded ahead
  auto load = [&](int r) {
    const Where w = where(r);
    if (wg_read) {
      const GC *p = T + w.base;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = threadIdx.x + u * NT;
        const int rr = min(e & (G - 1), w.L - 1), k = min(e >> lgG, n - 1);
        cur[u] = ldg(p + (k * stride + rr));
      }
    } else if (on) {
      const int b = line_base(w);
      const GC *p = (PASS == 0 ? X : T) + b;
#pragma unroll
      for (int q = 0; q < 8; ++q) cur[q] = ldg(p + team_idx(t, q));
    }
  };
  load(g0);
  for (int r = g0; r < g1; ++r) {
    const Where w = where(r);
    if (wg_read) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = threadIdx.x + u * NT, rr = e & (G - 1), k = e >> lgG;
        if (k < n) buf[rr * t.LS + swz<double>(k + 1)] = cur[u];
      }
      __syncthreads();
    } else if (on) {
#pragma unroll
      for (int q = 0; q < 8; ++q) lb[swz<double>(t.j + q * t.T)] = cur[q];
    }
    team_fresh(t);
    if (r + 1 < g1) load(r + 1);
    const bool act = t.g < w.L;   // L <= G
    if (on) {
      if constexpr (PASS == 2) {
        Cx<double> o[8];
        double mu[8];
        team_dst(lb, smem, t, o, false);
        team_mu0<double>(S, t, mu);
        const int l = min(w.l0 + t.g, lines - 1);
        double m1, m2 = 0.0;
        if (D == 2) {
          m1 = mode_mu<double>(S, 1)[l];
        } else {
          m1 = mode_mu<double>(S, 1)[l];
          m2 = mode_mu<double>(S, 2)[r / per];
        }
        team_sync(t);
        (void)team_scale<double>(S, lb, t, o, mu, act,
                                 [&](double m0) { return D == 2 ? m0 + m1 : (m0 + m1) + m2; });
      }
      if constexpr (wg_write) {
        team_dst_lds(lb, smem, t, PASS >= 2);
      } else {
        Cx<double> o[8];
        team_dst(lb, smem, t, o, PASS >= 2);
        GC *p = (PASS == 4 ? Y : T) + line_base(w);
        if (act) {
#pragma unroll
          for (int q = 0; q < 8; ++q)
            if (team_pt0(t, q) && (q < 4 || t.N > 4)) st_nt(p + team_idx(t, q), o[q]);
        }
        team_sync(t);
      }
    }
    if constexpr (wg_write) {
      __syncthreads();
      GC *p = T + w.base;
      for (int e = threadIdx.x; e < (n << lgG); e += NT) {
        const int rr = e & (G - 1), k = e >> lgG;
        if (rr < w.L) st_nt(p + (k * stride + rr), buf[rr * t.LS + swz<double>(k + 1)]);
      }
    }
    // the next round's values replace this one's lines
    if (wg_read || wg_write) __syncthreads();
  }
}

// Lines a round: a workgroup's, or as few as still leave a CU no more than one
// round, down to the eight that fill a 128-byte line of T (63^3: 38 us; halved
// until every CU has a round, and some have two, 51 us; always a workgroup's
// lines, 50 us).
template <int D, int PASS>
static hipError_t pass(const SysDesc *dsys, const SysDesc &h, int cus, const double2 *x, double2 *y,
                       hipStream_t s) {
  constexpr int ax = (PASS == 0 || PASS == 4) ? D - 1 : (PASS == 2 ? 0 : 1);
  const long long groups = D == 3 && ax == 0 ? h.n[2] : 1;
  const long long lines = groups > 1 ? h.n[1] : (ax == D - 1 ? h.rows : (long long)h.M / h.n[ax]);
  int lg = 31 - __builtin_clz(team_lines(h.n[ax]));
  auto rounds = [&](int l) { return groups * ((lines + (1 << l) - 1) >> l); };
  while (lg > 3 && rounds(lg - 1) <= cus) --lg;
  const int grid = (int)std::min<long long>(rounds(lg), cus);
  hipLaunchKernelGGL((pinv_team_kernel<D, PASS>), dim3(grid), dim3(NT), kTeamLds64Bytes, s, dsys, x, y, lg);
  return hipGetLastError();
}

hipError_t upload_twiddles(const double2 *tw64, const float2 *tw32) {
  hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(g_tw64), tw64, sizeof(double2) * TWN);
  if (e != hipSuccess) return e;
  return hipMemcpyToSymbol(HIP_SYMBOL(g_tw32), tw32, sizeof(float2) * TWN);
}

hipError_t launch_pinv(const SysDesc *dsys, const SysDesc &h, int cus, const double2 *x, double2 *y,
                       hipStream_t s) {
  hipError_t e;
  if (h.d == 2) {
    if ((e = pass<2, 0>(dsys, h, cus, x, y, s)) != hipSuccess) return e;
    if ((e = pass<2, 2>(dsys, h, cus, x, y, s)) != hipSuccess) return e;
    return pass<2, 4>(dsys, h, cus, x, y, s);
  }
  if ((e = pass<3, 0>(dsys, h, cus, x, y, s)) != hipSuccess) return e;
  if ((e = pass<3, 1>(dsys, h, cus, x, y, s)) != hipSuccess) return e;
  if ((e = pass<3, 2>(dsys, h, cus, x, y, s)) != hipSuccess) return e;
  if ((e = pass<3, 3>(dsys, h, cus, x, y, s)) != hipSuccess) return e;
  return pass<3, 4>(dsys, h, cus, x, y, s);
}

}  // namespace pinv512
}  // namespace csl

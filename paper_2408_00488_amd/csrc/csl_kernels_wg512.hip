// The persistent MINRES solver (arXiv:2408.00488) compiled for workgroups of
// 512 threads, namespace csl::wg512, for 2-D systems whose sine transforms all
// run as FFTs: the team phases (csl_team.hpp), one workgroup per CU.  At two
// waves a SIMD a wave has 256 registers (none spilled), so the operands of
// eight points are in flight per lane.  Two such workgroups per CU at 128
// registers run the phases no faster (a round of eight rows of 511 points in
// phase X 39 us for two against 20 us for one, batch of 64 systems of 63^2 to
// 511^2 points) and spill; the batch takes 22.0 ms there against 20.5 ms.
#define CSL_NT 512
#define CSL_KNS wg512
#define CSL_SOLVE_ONLY 1
#define CSL_2D_FFT_ONLY 1
#define CSL_TEAM 1
#define CSL_WAVES_PER_EU 2
#include "csl_kernels.hip"

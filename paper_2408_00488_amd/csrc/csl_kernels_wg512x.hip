// The persistent MINRES solver (arXiv:2408.00488) compiled for workgroups of
// 512 threads for systems of either dimension whose sine transforms all run
// as FFTs, namespace csl::wg512x: the team phases (csl_team.hpp) with the 3-D
// ones (5 per iteration), two workgroups per CU at 128 registers.  Its 3-D
// phases stream more than they compute, so the second workgroup pays here (a
// 255^3 solve 98 ms against 116 ms with one workgroup at 256 registers);
// batches of 2-D systems alone take csl::wg512.
#define CSL_NT 512
#define CSL_KNS wg512x
#define CSL_SOLVE_ONLY 1
#define CSL_FFT_ONLY 1
#define CSL_TEAM 1
#include "csl_kernels.hip"

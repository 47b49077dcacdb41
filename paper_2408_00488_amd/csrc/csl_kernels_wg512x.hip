// The persistent MINRES solver (arXiv:2408.00488) compiled for workgroups of
// 512 threads for systems of either dimension whose sine transforms all run
// as FFTs, namespace csl::wg512x: the team phases (csl_team.hpp) with the 3-D
// ones (5 per iteration), one workgroup per CU at 256 registers, none spilled
// (two at 128 spill 128: a 127^3 solve with the FP32 preconditioner 14.7 ms
// against 10.4 ms, 255^3 FP64 76.4 against 73.4 ms).  Batches of 2-D systems
// alone take csl::wg512.
#define CSL_NT 512
#define CSL_KNS wg512x
#define CSL_SOLVE_ONLY 1
#define CSL_FFT_ONLY 1
#define CSL_TEAM 1
#define CSL_WAVES_PER_EU 2
#include "csl_kernels.hip"

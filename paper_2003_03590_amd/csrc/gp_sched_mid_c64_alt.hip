// Axis-pass schedule variants for 64 .. 128 points, complex64 (autotuner alternatives).
#include "gp_registry.h"

GPK_SCHED(float, gpk::P_C64, 1, 64, 8, 16, 8, 8, 1)
GPK_SCHED(float, gpk::P_C64, 2, 64, 1, 64, 64, 1, 1)
GPK_SCHED(float, gpk::P_C64, 1, 96, 4, 16, 24, 4, 1)
GPK_SCHED(float, gpk::P_C64, 2, 96, 2, 32, 16, 6, 1)
GPK_SCHED(float, gpk::P_C64, 1, 128, 8, 8, 16, 8, 1)
GPK_SCHED(float, gpk::P_C64, 2, 128, 4, 16, 32, 4, 1)

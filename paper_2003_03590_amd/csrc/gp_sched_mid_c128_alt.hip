// Axis-pass schedule variants for 64 .. 128 points, complex128 (autotuner alternatives).
#include "gp_registry.h"

GPK_SCHED(double, gpk::P_C128, 1, 64, 4, 16, 16, 4, 1)
GPK_SCHED(double, gpk::P_C128, 1, 96, 4, 16, 24, 4, 1)
GPK_SCHED(double, gpk::P_C128, 1, 128, 8, 8, 8, 16, 1)
GPK_SCHED(double, gpk::P_C128, 2, 128, 8, 16, 16, 8, 1)

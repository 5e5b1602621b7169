// Axis-pass schedules for 256 points, complex128, and their variants (autotuner alternatives).
#include "gp_registry.h"

GPK_SCHED(double, gpk::P_C128, 0, 256, 16, 8, 16, 16, 1)
GPK_SCHED(double, gpk::P_C128, 1, 256, 16, 4, 16, 16, 1)
GPK_SCHED(double, gpk::P_C128, 2, 256, 16, 16, 16, 16, 1)
GPK_SCHED(double, gpk::P_C128, 3, 256, 32, 4, 8, 8, 4)

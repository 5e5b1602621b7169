// Axis-pass schedules for 256 points, complex64, and their variants (autotuner alternatives).
#include "gp_registry.h"

GPK_SCHED(float, gpk::P_C64, 0, 256, 16, 16, 16, 16, 1)
GPK_SCHED(float, gpk::P_C64, 1, 256, 16, 8, 16, 16, 1)
GPK_SCHED(float, gpk::P_C64, 2, 256, 8, 16, 32, 8, 1)
GPK_SCHED(float, gpk::P_C64, 3, 256, 16, 32, 16, 16, 1)

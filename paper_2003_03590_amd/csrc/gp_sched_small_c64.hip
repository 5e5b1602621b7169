// Axis-pass schedules for short axes (2 .. 48 points), complex64.
#include "gp_registry.h"

GPK_SCHED(float, gpk::P_C64, 0, 2, 1, 64, 2, 1, 1)
GPK_SCHED(float, gpk::P_C64, 0, 3, 1, 64, 3, 1, 1)
GPK_SCHED(float, gpk::P_C64, 0, 4, 1, 64, 4, 1, 1)
GPK_SCHED(float, gpk::P_C64, 0, 6, 1, 64, 6, 1, 1)
GPK_SCHED(float, gpk::P_C64, 0, 8, 1, 64, 8, 1, 1)
GPK_SCHED(float, gpk::P_C64, 0, 12, 1, 64, 12, 1, 1)
GPK_SCHED(float, gpk::P_C64, 0, 16, 1, 64, 16, 1, 1)
GPK_SCHED(float, gpk::P_C64, 0, 24, 1, 64, 24, 1, 1)
GPK_SCHED(float, gpk::P_C64, 0, 32, 2, 32, 16, 2, 1)
GPK_SCHED(float, gpk::P_C64, 0, 48, 2, 32, 24, 2, 1)

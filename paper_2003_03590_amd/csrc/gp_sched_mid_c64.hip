// Axis-pass schedules for 64 .. 192 points, complex64.
#include "gp_registry.h"

GPK_SCHED(float, gpk::P_C64, 0, 64, 4, 16, 16, 4, 1)
GPK_SCHED(float, gpk::P_C64, 0, 96, 4, 16, 12, 8, 1)
GPK_SCHED(float, gpk::P_C64, 0, 128, 8, 16, 16, 8, 1)
GPK_SCHED(float, gpk::P_C64, 0, 192, 8, 16, 24, 8, 1)

// Axis-pass schedules for 384 .. 1024 points, complex128.
#include "gp_registry.h"

GPK_SCHED(double, gpk::P_C128, 0, 384, 16, 8, 8, 8, 6)
GPK_SCHED(double, gpk::P_C128, 0, 512, 32, 8, 8, 8, 8)
GPK_SCHED(double, gpk::P_C128, 0, 768, 32, 4, 8, 8, 12)
GPK_SCHED(double, gpk::P_C128, 0, 1024, 64, 4, 16, 16, 4)

// Kernel launch with the optional timing events of the profiling aid.
#pragma once

#include <hip/hip_ext.h>

#include "pbd_kernels.h"

// With events set, kernels are launched with hipExtLaunchKernel, whose events
// carry the dispatch's own start and end times.
#define PBD_LAUNCH(KERNEL, GRID, BLOCK, SHMEM, ST, ...)                                              \
    do {                                                                                            \
        hipEvent_t _e0, _e1;                                                                        \
        pbd::get_launch_events(&_e0, &_e1);                                                         \
        if (_e0)                                                                                    \
            hipExtLaunchKernelGGL(KERNEL, GRID, BLOCK, SHMEM, ST, _e0, _e1, 0, __VA_ARGS__);        \
        else                                                                                        \
            hipLaunchKernelGGL(KERNEL, GRID, BLOCK, SHMEM, ST, __VA_ARGS__);                        \
    } while (0)

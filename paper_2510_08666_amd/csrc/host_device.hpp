// For rules that both the host and the kernels follow, in headers that the host compiler takes as well.
#pragma once

#if defined(__HIPCC__)
#define DINFER_HOST_DEVICE __host__ __device__
#else
#define DINFER_HOST_DEVICE
#endif

// Host stand-ins for the HIP types that the kernel sources' host code names.
#pragma once
#include <stddef.h>
#include <stdint.h>

#define __device__
#define __host__
typedef int hipError_t;
typedef void *hipStream_t, *hipEvent_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidConfiguration = 9, hipErrorUnknown = 999 };
enum { hipMemcpyDeviceToHost, hipMemcpyHostToDevice };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }

// Stand-in for the HIP runtime's host interface, as far as csrc/lc_api.hip uses it, for a host-only build of that file:
// host_failures.cpp defines the functions and lets them fail on demand.
#pragma once
#include <stddef.h>

#define __host__
#define __device__
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) (&(x))

enum hipError_t { hipSuccess = 0, hipErrorUnknown = 999 };
struct FakeStream;
struct FakeEvent;
typedef FakeStream* hipStream_t;
typedef FakeEvent* hipEvent_t;
enum { hipEventDisableTiming = 2, hipHostMallocDefault = 0, hipHostMallocPortable = 1, hipHostMallocMapped = 2 };

hipError_t hipGetDevice(int* dev);
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags);
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s);
hipError_t hipEventSynchronize(hipEvent_t e);
hipError_t hipStreamSynchronize(hipStream_t s);
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned flags);
hipError_t hipHostFree(void* p);
hipError_t hipGetSymbolAddress(void** p, const void* symbol);
const char* hipGetErrorString(hipError_t e);

// The part of the HIP runtime's interface that the library's host code uses,
// for builds of that code with g++ (api_host.cpp): "device" memory is host
// memory, streams run nothing, and allocations can be made to fail.
#pragma once

#include <stddef.h>
#include <stdint.h>

#define __device__
#define __align__(x) __attribute__((aligned(x)))
#define HIP_SYMBOL(x) ((const void *)&(x))

enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2 };
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };
typedef struct stubStream *hipStream_t;
typedef struct stubEvent *hipEvent_t;
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount = 63 };
constexpr unsigned hipStreamNonBlocking = 1, hipEventDisableTiming = 2;

const char *hipGetErrorString(hipError_t);
hipError_t hipGetLastError();
hipError_t hipMalloc(void **p, size_t bytes);
hipError_t hipFree(void *p);
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned flags = 0);
hipError_t hipHostFree(void *p);
hipError_t hipMemGetInfo(size_t *free_bytes, size_t *total);
hipError_t hipMemcpy(void *to, const void *from, size_t bytes, hipMemcpyKind);
hipError_t hipMemcpyAsync(void *to, const void *from, size_t bytes, hipMemcpyKind, hipStream_t);
hipError_t hipMemsetAsync(void *p, int value, size_t bytes, hipStream_t);
hipError_t hipGetSymbolAddress(void **p, const void *symbol);
hipError_t hipGetDevice(int *device);
hipError_t hipSetDevice(int device);
hipError_t hipDeviceGetAttribute(int *value, hipDeviceAttribute_t, int device);
hipError_t hipDeviceSynchronize();
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned flags);
hipError_t hipStreamDestroy(hipStream_t);
hipError_t hipStreamSynchronize(hipStream_t);
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned flags);
hipError_t hipEventCreate(hipEvent_t *e);
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned flags);
hipError_t hipEventDestroy(hipEvent_t);
hipError_t hipEventRecord(hipEvent_t, hipStream_t);
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t);

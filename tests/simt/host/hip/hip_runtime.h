// Stands in for <hip/hip_runtime.h> when the library's host code is compiled
// with g++ (tests only): the runtime calls that code makes, over the device of
// device.cpp.
#pragma once

#include <cstddef>
#include <cstdint>
#include <mutex>

enum hipError_t {
  hipSuccess = 0,
  hipErrorOutOfMemory = 2,
  hipErrorMemoryAllocation = 2,
  hipErrorInvalidValue = 1,
  hipErrorNotReady = 600,
  hipErrorLaunchTimeOut = 702,
  hipErrorUnknown = 999
};
typedef struct SimStream* hipStream_t;
typedef struct SimEvent* hipEvent_t;
typedef struct SimGraph* hipGraph_t;
typedef struct SimGraph* hipGraphExec_t;
struct hipDeviceProp_t {
  int multiProcessorCount;
  size_t sharedMemPerBlock, maxSharedMemoryPerMultiProcessor;
  char gcnArchName[32];
};
enum hipMemoryType { hipMemoryTypeHost, hipMemoryTypeDevice, hipMemoryTypeManaged };
struct hipPointerAttribute_t {
  hipMemoryType type;
};
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum { hipStreamNonBlocking = 1, hipEventDisableTiming = 2, hipHostMallocDefault = 0, hipHostMallocCoherent = 1,
       hipHostMallocMapped = 2 };
enum hipStreamCaptureMode { hipStreamCaptureModeThreadLocal };
enum hipDeviceAttribute_t { hipDeviceAttributeWallClockRate };

hipError_t hipGetDeviceCount(int*);
hipError_t hipGetDevice(int*);
hipError_t hipSetDevice(int);
hipError_t hipGetDeviceProperties(hipDeviceProp_t*, int);
hipError_t hipDeviceGetAttribute(int*, hipDeviceAttribute_t, int);
const char* hipGetErrorString(hipError_t);
hipError_t hipGetLastError();
hipError_t sim_malloc(void**, size_t);
template <class T>
hipError_t hipMalloc(T** p, size_t n) { return sim_malloc(reinterpret_cast<void**>(p), n); }
hipError_t hipFree(void*);
hipError_t sim_host_malloc(void**, size_t);
template <class T>
hipError_t hipHostMalloc(T** p, size_t n, unsigned) { return sim_host_malloc(reinterpret_cast<void**>(p), n); }
hipError_t hipHostFree(void*);
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind);
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t);
hipError_t hipMemset(void*, int, size_t);
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t);
hipError_t hipPointerGetAttributes(hipPointerAttribute_t*, const void*);
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned);
hipError_t hipStreamDestroy(hipStream_t);
hipError_t hipStreamQuery(hipStream_t);
hipError_t hipStreamSynchronize(hipStream_t);
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned);
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode);
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*);
hipError_t hipEventCreate(hipEvent_t*);
hipError_t hipEventCreateWithFlags(hipEvent_t*, unsigned);
hipError_t hipEventDestroy(hipEvent_t);
hipError_t hipEventRecord(hipEvent_t, hipStream_t);
hipError_t hipEventQuery(hipEvent_t);
hipError_t hipEventSynchronize(hipEvent_t);
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t);
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, void*, char*, size_t);
hipError_t hipGraphDestroy(hipGraph_t);
hipError_t hipGraphExecDestroy(hipGraphExec_t);
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t);

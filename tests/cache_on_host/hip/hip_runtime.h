// What zipmoe_cache.hip needs of the HIP runtime, for its build as ordinary host code: "device" memory is process memory,
// copies and launches run at once, and the process keeps a list of what a kernel could reach and of what a real
// runtime could still have under way.  cache_on_host.cpp has the
// definitions.
#pragma once
#include <cstddef>
#include <cstdint>

#define __global__
#define __launch_bounds__(...)

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorNotFound = 500, hipErrorCapturedEvent = 907 };
enum hipMemoryType { hipMemoryTypeUnregistered = 0, hipMemoryTypeHost = 1, hipMemoryTypeDevice = 2, hipMemoryTypeManaged = 3 };
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToDevice = 3 };
constexpr unsigned hipStreamNonBlocking = 1, hipEventDisableTiming = 2;
typedef struct fake_stream *hipStream_t;
typedef struct fake_event *hipEvent_t;
typedef void *hipDeviceptr_t;
struct hipPointerAttribute_t {
    hipMemoryType type;
    int device;
    void *devicePointer, *hostPointer;
    int isManaged;
    unsigned allocationFlags;
};
struct dim3 {
    uint32_t x, y, z;
    dim3(uint32_t x_ = 1, uint32_t y_ = 1, uint32_t z_ = 1) : x(x_), y(y_), z(z_) {}
};
extern thread_local dim3 blockIdx, threadIdx;

hipError_t hipPointerGetAttributes(hipPointerAttribute_t *attributes, const void *p);
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t p);
hipError_t hipGetLastError();
hipError_t hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream);
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t bytes, hipMemcpyKind kind, hipStream_t stream);
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone = 0, hipStreamCaptureStatusActive = 1 };
hipError_t hipStreamCreateWithFlags(hipStream_t *stream, unsigned flags);
hipError_t hipStreamSynchronize(hipStream_t stream);
hipError_t hipStreamWaitEvent(hipStream_t stream, hipEvent_t event, unsigned flags);
hipError_t hipStreamIsCapturing(hipStream_t stream, hipStreamCaptureStatus *status);
hipError_t hipEventCreateWithFlags(hipEvent_t *event, unsigned flags);
hipError_t hipEventRecord(hipEvent_t event, hipStream_t stream);
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }

// What csrc/path_a.cpp uses of HIP, for a host program that plays the device (host_path_a.cpp).
#pragma once
#include <cstddef>
typedef int hipError_t;
typedef void* hipStream_t;
enum { hipSuccess = 0, hipErrorUnknown = 999 };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeRelaxed };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum { hipHostMallocPortable = 1, hipHostMallocMapped = 2, hipHostMallocCoherent = 4 };
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags);
hipError_t hipHostFree(void* p);
hipError_t hipGetLastError();
hipError_t hipStreamSynchronize(hipStream_t st);
hipError_t hipStreamIsCapturing(hipStream_t st, hipStreamCaptureStatus* status);
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* mode);
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t st);
hipError_t hipMemcpyWithStream(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t st);

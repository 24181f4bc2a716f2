// aes_launch.hpp -- the launch of one kernel with its arguments in one block.
//
// A launch through the kernel's host symbol costs the calling thread 4.0 us
// with the 264 bytes of an ECB call's arguments (round keys by value); with
// the device function looked up once and the arguments copied as one block,
// laid out as the kernel reads them, 3.1 us.  A small buffer's call is bound
// by that, not by the 2.5-4 us its kernel runs.
#pragma once
#include <hip/hip_runtime.h>
#include <atomic>
#include <cstddef>
#include <cstdint>
#include <cstring>

namespace aesgpu {

template <class T>
struct AsIs {
    using type = T;
};

// The kernel's function on the device of `stream`, looked up on its first
// launch there (null if it cannot be: more devices than the table, or a
// runtime that refuses).
template <auto K>
hipFunction_t kernel_function(hipStream_t stream)
{
    static std::atomic<hipFunction_t> known[64];
    int current = -1, dev = -1;
    if (hipGetDevice(&current) != hipSuccess)
        return nullptr;
    dev = current;
    if (stream != nullptr && hipStreamGetDevice(stream, &dev) != hipSuccess)
        return nullptr;
    if (dev < 0 || dev >= 64)
        return nullptr;
    hipFunction_t f = known[dev].load(std::memory_order_acquire);
    if (f == nullptr && dev == current && hipGetFuncBySymbol(&f, reinterpret_cast<const void*>(K)) == hipSuccess)
        known[dev].store(f, std::memory_order_release);
    return f;
}

// Arguments at their natural alignment, one after the other: the kernel
// argument block of the device ABI.
template <class T>
void pack_argument(unsigned char* block, size_t& at, const T& v)
{
    at = (at + alignof(T) - 1) / alignof(T) * alignof(T);
    std::memcpy(block + at, &v, sizeof(T));
    at += sizeof(T);
}

template <auto K, class... P>
hipError_t launch_packed(void (*)(P...), unsigned grid, unsigned wg, hipStream_t stream,
                         typename AsIs<P>::type... args)
{
    if (hipFunction_t f = kernel_function<K>(stream)) {
        alignas(16) unsigned char block[(0u + ... + (sizeof(P) + alignof(P)))];
        size_t size = 0;
        (pack_argument<P>(block, size, args), ...);
        void* extra[] = {HIP_LAUNCH_PARAM_BUFFER_POINTER, block, HIP_LAUNCH_PARAM_BUFFER_SIZE, &size,
                         HIP_LAUNCH_PARAM_END};
        const hipError_t e = hipModuleLaunchKernel(f, grid, 1, 1, wg, 1, 1, 0, stream, nullptr, extra);
        if (e != hipSuccess)
            (void)hipGetLastError();  // reported here, not by the next launch
        return e;
    }
    (void)hipGetLastError();
    K<<<dim3(grid), dim3(wg), 0, stream>>>(args...);
    return hipGetLastError();
}

// Enqueue kernel K with `grid` workgroups of `wg` threads.
template <auto K, class... A>
hipError_t launch_kernel(unsigned grid, unsigned wg, hipStream_t stream, A... args)
{
    return launch_packed<K>(K, grid, wg, stream, args...);
}

}  // namespace aesgpu

// Kernel launches as data.  A launcher calls launch(kernel, grid, block, lds, stream, args...): on a thread that has a
// recorder the launch is written down (kernel, grid, packed arguments) instead of being made, which is how a schedule
// turns into queue packets (lanes.h); without one it is an ordinary launch on the HIP stream.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <tuple>
#include <type_traits>
#include <vector>

namespace mt {

class LaneDevice;

// What a dispatch packet has to say about a kernel (read from the loaded code object).
struct KernelCode {
    uint64_t object = 0;                 // address of the kernel descriptor
    uint32_t kernarg_bytes = 0, group_bytes = 0, private_bytes = 0;
};

struct RecordedLaunch {
    const KernelCode *code;
    uint32_t grid[3];                    // workgroups
    uint32_t block[3];
    uint32_t dyn_lds;
    size_t arg_off, arg_bytes;           // explicit arguments inside LaunchRecorder::args
};

struct LaunchRecorder {
    LaneDevice *dev = nullptr;
    std::vector<RecordedLaunch> launches;
    std::vector<uint8_t> args;
    int walked = 0, deep = 0;            // launches cut to a share of the units, and staged deep (mt_schedule_launch_forms)
    int error = 0;                       // hipError_t of the first launch that could not be written down
    void add(const void *host_fn, dim3 grid, dim3 block, size_t lds, const void *packed, size_t bytes);
};

LaunchRecorder *&current_recorder();     // of the calling thread, null = launch for real

inline void count_launch(int LaunchRecorder::*what) {
    if (LaunchRecorder *r = current_recorder()) ++(r->*what);
}

template <typename... P, typename... A>
inline void launch(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t st, const A &...args) {
    static_assert(sizeof...(P) == sizeof...(A), "one value per kernel parameter");
    if (LaunchRecorder *r = current_recorder()) {
        constexpr size_t room = (0 + ... + (sizeof(P) + alignof(P)));
        alignas(16) unsigned char buf[room];
        size_t off = 0;
        auto put = [&]<typename Q>(const Q &v) {
            off = (off + alignof(Q) - 1) / alignof(Q) * alignof(Q);
            std::memcpy(buf + off, &v, sizeof(Q));
            off += sizeof(Q);
        };
        (put(static_cast<std::remove_cv_t<P>>(args)), ...);
        r->add((const void *)kernel, grid, block, lds, buf, off);
    } else {
        std::tuple<std::remove_cv_t<P>...> values(args...);
        std::apply([&](auto &...v) {
            void *ptrs[] = {(void *)&v...};
            (void)hipLaunchKernel((const void *)kernel, grid, block, ptrs, lds, st);
        }, values);
    }
}

}  // namespace mt

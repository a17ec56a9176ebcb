// Launchers of the wavefront forward kernels.  Each geometry (rows per lane
// R, lanes per stream LS, traceback / end-cell variant, profile width) is a
// separate template instance; the instances are spread over several
// translation units (launch_stream_*.hip) so that they compile in parallel.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stddef.h>

#include "sw_kernels.hpp"

namespace hk {

// Events that take a kernel's own start and end times (null: none).  Recorded
// with the dispatch, they cost nothing on the stream; hipEventRecord between
// kernels left a gap of 5.6 us at each.
struct Timed {
    hipEvent_t start = nullptr, stop = nullptr;
};
template <typename K, typename... A>
void launch_timed(const Timed &t, K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t st, A... args) {
    if (t.start || t.stop) hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, st, t.start, t.stop, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, st, args...);
}

// 64-lane streams with R = 1..8 (int16 or int32 profile); 32- and 16-lane
// streams with R = 2..16 (int16 profile)
inline bool stream_supported(int R, int LS, bool p16) {
    if (LS == 64) return R >= 1 && R <= 8;
    return (LS == 32 || LS == 16) && p16 && R >= 2 && R <= 16;
}

// packed 16-bit kernel (end cells, with or without traceback): 32- and 16-lane streams, R = 2..16
inline bool stream16_supported(int R, int LS) { return (LS == 32 || LS == 16) && R >= 2 && R <= 16; }

// sw_stream_kernel for R in [1, 5], [6, 10] and [11, 16] (one translation unit each)
void launch_stream_r1(int R, int LS, const StreamArgs &a, bool tb, bool endc, bool p16, int grid, int threads, size_t lds,
                      hipStream_t st, const Timed &t);
void launch_stream_r6(int R, int LS, const StreamArgs &a, bool tb, bool endc, bool p16, int grid, int threads, size_t lds,
                      hipStream_t st, const Timed &t);
void launch_stream_r11(int R, int LS, const StreamArgs &a, bool tb, bool endc, bool p16, int grid, int threads, size_t lds,
                       hipStream_t st, const Timed &t);
// sw_stream16_kernel for R in [2, 9] and [10, 16]
void launch_stream16_r2(int R, int LS, const StreamArgs &a, bool tb, int grid, int threads, size_t lds, hipStream_t st,
                        const Timed &t);
void launch_stream16_r10(int R, int LS, const StreamArgs &a, bool tb, int grid, int threads, size_t lds, hipStream_t st,
                         const Timed &t);

inline void launch_stream(int R, int LS, const StreamArgs &a, bool tb, bool endc, bool p16, int grid, int threads, size_t lds,
                          hipStream_t st, const Timed &t) {
    if (R <= 5) launch_stream_r1(R, LS, a, tb, endc, p16, grid, threads, lds, st, t);
    else if (R <= 10) launch_stream_r6(R, LS, a, tb, endc, p16, grid, threads, lds, st, t);
    else launch_stream_r11(R, LS, a, tb, endc, p16, grid, threads, lds, st, t);
}

inline void launch_stream16(int R, int LS, const StreamArgs &a, bool tb, int grid, int threads, size_t lds,
                            hipStream_t st, const Timed &t) {
    if (R <= 9) launch_stream16_r2(R, LS, a, tb, grid, threads, lds, st, t);
    else launch_stream16_r10(R, LS, a, tb, grid, threads, lds, st, t);
}

}  // namespace hk

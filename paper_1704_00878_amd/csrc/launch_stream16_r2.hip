// sw_stream16_kernel (packed 16-bit) instances with R = 2..9 rows per lane.
#include "launch_stream_impl.hpp"

namespace hk {

void launch_stream16_r2(int R, int LS, const StreamArgs &a, bool tb, int grid, int threads, size_t lds, hipStream_t st, const Timed &t) {
    launch_stream16_range<2, 9>(R, LS, a, tb, grid, threads, lds, st, t);
}

}  // namespace hk

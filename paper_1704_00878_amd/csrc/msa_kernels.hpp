// Center-star merge and row emission (Fig. 3: the first reduction builds the
// longest center-star sequence from all inserted-space vectors; the second map
// builds each row from its inserted-space vector and its own sequence), plus
// encoding, small fills and the avg SP evaluation of the Results section.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hk {

constexpr int kGap = 255;

// Fill with a kernel (graph-capturable, no memset nodes).
__global__ void fill_u32_kernel(uint32_t *p, uint32_t v, int64_t n) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n;
         x += (int64_t)gridDim.x * blockDim.x)
        p[x] = v;
}

// A substitution matrix passed by value (kernel argument), copied into device
// memory by one workgroup: no host staging buffer is involved.
struct MatrixArg {
    int8_t v[32 * 32];
};

__global__ void matrix_copy_kernel(MatrixArg mat, int n, int8_t *dst) {
    for (int x = threadIdx.x; x < n; x += blockDim.x) dst[x] = mat.v[x];
}

// Score-only calls that ask for cells report (0, 0, i1, j1).
__global__ void endcell_to_cells_kernel(const int32_t *endcell, int n, int32_t *cells) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    reinterpret_cast<int4 *>(cells)[k] = make_int4(0, 0, endcell[2 * k], endcell[2 * k + 1]);
}

// Largest code in [p, p + n), 16-byte loads where aligned.
__device__ __forceinline__ int maxcode_range(const uint8_t *p, int64_t n, int64_t tid, int64_t stride) {
    int mx = 0;
    const int64_t head = min<int64_t>(n, (int64_t)((16 - ((uintptr_t)p & 15)) & 15));
    for (int64_t x = tid; x < head; x += stride) mx = max(mx, (int)p[x]);
    const int64_t nv = (n - head) >> 4;
    const uint4 *pv = reinterpret_cast<const uint4 *>(p + head);
    for (int64_t x = tid; x < nv; x += stride) {
        const uint4 v = pv[x];
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int y = 0; y < 4; ++y)
            mx = max(mx, max(max((int)(w[y] & 255), (int)((w[y] >> 8) & 255)),
                             max((int)((w[y] >> 16) & 255), (int)(w[y] >> 24))));
    }
    for (int64_t x = head + (nv << 4) + tid; x < n; x += stride) mx = max(mx, (int)p[x]);
    return mx;
}

// What a call does before its first real kernel, in one launch: up to four word
// ranges (and one trailing uint16) zeroed; the largest code of two ranges raised
// into *out as (tag | code) with atomicMax, one atomic per workgroup; the score
// matrix fetched from pinned host memory; and, by the last hwgs workgroups, the
// pairs counted by length, each into a row of hpart.  Apart, each cost its launch
// (5 us at 64 pairs, whose kernels wait for the host) and the copy 8 us.
struct PrepArgs {
    uint32_t *z[4];
    int64_t nz[4];
    uint16_t *tail16;
    const uint8_t *p, *q;
    int64_t n, nq;
    uint32_t tag, *out;
    const uint32_t *msrc;
    uint32_t *mdst;
    int mwords;
    const int64_t *off;
    int np, maxlen, hwgs;
    int32_t *hpart;           // [hwgs][maxlen + 1]
};
constexpr int kPrepHistMax = 4096;   // lengths counted there

__global__ void __launch_bounds__(256) prep_kernel(PrepArgs a) {
    extern __shared__ int32_t s_hist[];   // [maxlen + 1] where pairs are counted
    __shared__ int red[4];
    const int t = threadIdx.x, wgs = gridDim.x - a.hwgs;
    if ((int)blockIdx.x >= wgs) {
        const int b = blockIdx.x - wgs;
        for (int x = t; x <= a.maxlen; x += 256) s_hist[x] = 0;
        __syncthreads();
        for (int x = b * 256 + t; x < a.np; x += a.hwgs * 256)
            atomicAdd(s_hist + (int)min<int64_t>(a.maxlen, a.off[x + 1] - a.off[x]), 1);
        __syncthreads();
        for (int x = t; x <= a.maxlen; x += 256) a.hpart[b * (a.maxlen + 1) + x] = s_hist[x];
        return;
    }
    const int64_t tid = (int64_t)blockIdx.x * 256 + t, stride = (int64_t)wgs * 256;
    if (tid < a.mwords) a.mdst[tid] = a.msrc[tid];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        uint32_t *z = a.z[r];
        const int64_t n = a.nz[r], n4 = ((uintptr_t)z & 15) == 0 ? n >> 2 : 0;
        for (int64_t x = tid; x < n4; x += stride) reinterpret_cast<uint4 *>(z)[x] = make_uint4(0u, 0u, 0u, 0u);
        for (int64_t x = 4 * n4 + tid; x < n; x += stride) z[x] = 0u;
    }
    if (tid == 0 && a.tail16) *a.tail16 = 0;
    if (a.n + a.nq <= 0) return;
    int mx = a.n > 0 ? maxcode_range(a.p, a.n, tid, stride) : 0;
    if (a.nq > 0) mx = max(mx, maxcode_range(a.q, a.nq, tid, stride));
    for (int sh = 32; sh > 0; sh >>= 1) mx = max(mx, __shfl_xor(mx, sh));
    if ((t & 63) == 0) red[t >> 6] = mx;
    __syncthreads();
    if (t == 0) atomicMax(a.out, a.tag | (uint32_t)max(max(red[0], red[1]), max(red[2], red[3])));
}

// ASCII -> residue code through a 256-entry table.
__global__ void encode_kernel(const uint8_t *ascii, int64_t len, uint8_t *codes, const uint8_t *table) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < len;
         x += (int64_t)gridDim.x * blockDim.x)
        codes[x] = table[ascii[x]];
}

// G[p] = max_k ins[k][p].  Block (256 threads) covers 256 slots x kRows rows,
// reduces in registers and publishes with one integer atomicMax per slot
// (max is order-independent, so the result is deterministic).
constexpr int kMergeRows = 64;
__global__ void merge_max_kernel(const uint16_t *ins, int n, int m1, int32_t *G) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= m1) return;
    const int k0 = blockIdx.y * kMergeRows;
    const int k1 = min(n, k0 + kMergeRows);
    int g = 0;
    for (int k = k0; k < k1; ++k) g = max(g, (int)ins[(int64_t)k * m1 + p]);
    if (g > 0) atomicMax(G + p, g);
}

// col[p] = sum_{q<p} (G[q] + 1); width = m + sum G.  One workgroup of 1024.
// mail (optional, host memory mapped for the device): mail[0] = width, then
// mail[1] = seq with a system-scope release, so a host spinning on mail[1]
// reads the width (and, in mail[2], the flag word) without a stream
// synchronisation
//
// Tiles of 4,096 positions, four per lane, the next tile's loads in flight while
// one is summed (32-bit sums fit a tile: 4,096 x 65,536), one barrier each.
// At 16,570 positions 21.5 us with a contiguous run per lane.
__global__ void __launch_bounds__(1024) merge_scan_kernel(const int32_t *G, int m1, int64_t *col, int64_t *width,
                                                          int64_t *mail, int64_t seq, const uint32_t *flag) {
    __shared__ int s_sum[2][16];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int nx[4];
    auto load = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int p = t0 + 4 * tid + u;
            nx[u] = p < m1 ? G[p] + 1 : 0;
        }
    };
    int64_t base = 0;   // of the tile
    load(0);
    int b = 0;
    for (int t0 = 0; t0 < m1; t0 += 4096, b ^= 1) {
        int v[4], sum = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[u] = nx[u];
            sum += v[u];
        }
        load(t0 + 4096);
        int inc = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(inc, d, 64);
            if (lane >= d) inc += t;
        }
        if (lane == 63) s_sum[b][wv] = inc;
        __syncthreads();   // (the other buffer is still being read by late wavefronts)
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int x = s_sum[b][w];
            before += w < wv ? x : 0;
            all += x;
        }
        int64_t acc = base + before + inc - sum;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int p = t0 + 4 * tid + u;
            if (p < m1) col[p] = acc;
            acc += v[u];
        }
        base += all;
    }
    if (tid == 0) {
        *width = base - 1;
        if (mail) {
            __hip_atomic_store(mail, base - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            if (flag) __hip_atomic_store(mail + 2, (int64_t)*flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(mail + 1, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// Rows: one wavefront per row, up to four wavefronts per workgroup, each
// with its own LDS region.  A row's insertion counts, aligned bits and residues
// are staged in LDS as aligned words, loaded while the row before is built;
// then the row is built in LDS a chunk of columns at a time: filled with
// gaps, its blocks shared by the lanes (a wave-wide prefix sum of their
// residues gives each lane its first one), and copied out with 16-byte stores.
// Block p's insertion t goes to column col[p] + t, its aligned residue to the center
// column col[p] + G[p]; blocks with more than kRowFew insertions (the ends of
// a local alignment) are placed by the whole wavefront.  The chunk sits in LDS at the
// row's misalignment, so aligned LDS words map onto aligned global words.
//
// Bound by latency: with the loads in line, a binary search per lane and each
// residue read from memory where it was placed, 20,000 rows of 311 + 1 blocks and
// 4,208 columns took 67 us, 300,000 of 200 + 1 and 5,015 902 us; now 43 and 535
// (2.8 TB/s of bytes written).
constexpr int kWaveRows = 4;
constexpr int kRowFew = 4;
constexpr int kRowPre = 4;        // aligned words per lane of counts and of residues loaded a row ahead
typedef uint16_t __attribute__((may_alias)) row_count_t;   // half of a staged word

struct RowsArgs {
    const uint8_t *res;
    const int64_t *off;
    int nrows, m;
    const uint16_t *ins;
    const uint32_t *aligned;
    int aw;
    const int32_t *G;         // [m+1]
    const int64_t *col;       // [m+1]
    int64_t width;
    int ch;                   // columns per chunk (multiple of 16)
    int wave_bytes;           // LDS bytes per wavefront region
    int res_bytes;            // residues of a row staged there at most (longer rows are read from memory)
    int gc_lds;               // col staged in LDS for the workgroup (after the wave regions)
    uint8_t *msa;             // [nrows][width]
};
__host__ __device__ inline size_t rows_ins_bytes(int m1) { return (2 * (size_t)m1 + 4 + 15) & ~(size_t)15; }
__host__ __device__ inline size_t rows_bit_bytes(int aw) { return (4 * (size_t)aw + 15) & ~(size_t)15; }

__global__ void __launch_bounds__(64 * kWaveRows) rows_kernel(RowsArgs a) {
    extern __shared__ uint4 lds_rows[];
    const int tid = threadIdx.x, wid = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wpb = blockDim.x >> 6;
    const int m = a.m, m1 = m + 1;
    const int64_t width = a.width;
    // per wavefront: insertion counts (uint16), aligned bits, residues, then
    // the row chunk [ch + 16]
    char *wsh = reinterpret_cast<char *>(lds_rows) + (size_t)wid * a.wave_bytes;
    uint32_t *iw = reinterpret_cast<uint32_t *>(wsh);
    uint32_t *abit = reinterpret_cast<uint32_t *>(wsh + rows_ins_bytes(m1));
    uint32_t *rw = abit + rows_bit_bytes(a.aw) / 4;
    uint8_t *buf = reinterpret_cast<uint8_t *>(rw) + a.res_bytes + 16;
    uint4 *buf16 = reinterpret_cast<uint4 *>(buf);
    // the workgroup's column table: col[p] for p <= m and width + 1 after
    // it, so block p's gap count is col[p + 1] - col[p] - 1
    int *gcl = reinterpret_cast<int *>(reinterpret_cast<char *>(lds_rows) + (size_t)wpb * a.wave_bytes);
    if (a.gc_lds) {
        for (int p = tid; p <= m1; p += blockDim.x) gcl[p] = p < m1 ? (int)a.col[p] : (int)(width + 1);
        __syncthreads();
    }
    auto colg = [&](int p) __attribute__((always_inline)) -> int2 {
        return a.gc_lds ? make_int2(gcl[p], gcl[p + 1] - gcl[p] - 1) : make_int2((int)a.col[p], a.G[p]);
    };
    auto colv = [&](int p) __attribute__((always_inline)) -> int {   // col[p], p <= m (below 2^31)
        return a.gc_lds ? gcl[p] : (int)a.col[p];
    };
    // a row's words: counts (from the aligned word that holds the first one),
    // residues (likewise), aligned bits
    struct Row {
        int64_t so;
        int n, iodd, rodd, ni, nr;   // words of counts and of residues
        const uint32_t *ip, *rp, *ap;
    };
    auto row_at = [&](int k, int64_t so, int64_t eo) __attribute__((always_inline)) {
        Row r;
        r.so = so;
        r.n = (int)(eo - so);
        const uintptr_t ia = (uintptr_t)(a.ins + (int64_t)k * m1), ra = (uintptr_t)(a.res + so);
        r.iodd = (int)(ia & 3) >> 1;
        r.rodd = (int)(ra & 3);
        r.ip = reinterpret_cast<const uint32_t *>(ia & ~(uintptr_t)3);
        r.rp = reinterpret_cast<const uint32_t *>(ra & ~(uintptr_t)3);
        r.ap = a.aligned + (int64_t)k * a.aw;
        r.ni = (r.iodd + m1 + 1) >> 1;
        r.nr = r.n > 0 && r.n <= a.res_bytes ? (r.rodd + r.n + 3) >> 2 : 0;
        return r;
    };
    const int step = gridDim.x * wpb;
    int k = blockIdx.x * wpb + wid;
    if (k >= a.nrows) return;
    uint32_t pi[kRowPre], pr[kRowPre], pa0 = 0;
    auto fetch = [&](const Row &r) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kRowPre; ++u) {
            const int i = 64 * u + lane;
            pi[u] = i < r.ni ? r.ip[i] : 0u;
            pr[u] = i < r.nr ? r.rp[i] : 0u;
        }
        pa0 = lane < a.aw ? r.ap[lane] : 0u;
    };
    Row r = row_at(k, a.off[k], a.off[k + 1]);
    fetch(r);
    int64_t no = 0, ne = 0;   // the next row's residues
    if (k + step < a.nrows) {
        no = a.off[k + step];
        ne = a.off[k + step + 1];
    }
    for (;;) {
        __builtin_amdgcn_wave_barrier();   // the previous row is done with this region
#pragma unroll
        for (int u = 0; u < kRowPre; ++u) {
            const int i = 64 * u + lane;
            if (i < r.ni) iw[i] = pi[u];
            if (i < r.nr) rw[i] = pr[u];
        }
        if (lane < a.aw) abit[lane] = pa0;
        // what a long center or row has past the prefetched words
        for (int i0 = 64 * kRowPre; i0 < r.ni || i0 < r.nr; i0 += 256) {
            uint32_t v[4], w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + 64 * u + lane;
                v[u] = i < r.ni ? r.ip[i] : 0u;
                w[u] = i < r.nr ? r.rp[i] : 0u;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + 64 * u + lane;
                if (i < r.ni) iw[i] = v[u];
                if (i < r.nr) rw[i] = w[u];
            }
        }
        for (int q = 64 + lane; q < a.aw; q += 64) abit[q] = r.ap[q];
        // other lanes read what this one staged (the wavefront's LDS accesses
        // stay in order once the compiler keeps them so)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const row_count_t *sins = reinterpret_cast<const row_count_t *>(iw) + r.iodd;
        const uint8_t *sres = reinterpret_cast<const uint8_t *>(rw) + r.rodd, *gres = a.res + r.so;
        const bool rl = r.n <= a.res_bytes;
        const int n = r.n;
        uint8_t *row = a.msa + (int64_t)k * width;
        const int a0 = (int)((uintptr_t)row & 15);
        const bool more = k + step < a.nrows;
        if (more) {   // the next row's words, and the offsets after it
            k += step;
            r = row_at(k, no, ne);
            fetch(r);
            if (k + step < a.nrows) {
                no = a.off[k + step];
                ne = a.off[k + step + 1];
            }
        }
        auto count = [&](int p) __attribute__((always_inline)) -> int {   // residues of block p
            return (int)sins[p] + (p < m ? (int)((abit[p >> 5] >> (p & 31)) & 1u) : 0);
        };
        int pa = 0, qa = 0;   // first block of the chunk, its first residue
        for (int64_t x0 = 0; x0 < width; x0 += a.ch) {
            const int len = (int)min<int64_t>(a.ch, width - x0), x1 = (int)x0 + len;
            int pe = m1;      // blocks with a column before x1: [pa, pe)
            if (x1 < width) {
                int lo = pa, hi = m1;   // the first block from x1 on
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (colv(mid) < x1) lo = mid + 1;
                    else hi = mid;
                }
                pe = lo;
            }
            const int nw = (a0 + len + 15) >> 4;
            for (int q = lane; q < nw; q += 64) buf16[q] = make_uint4(~0u, ~0u, ~0u, ~0u);
            const int per = (pe - pa + 63) >> 6;
            const int lo = min(pe, pa + lane * per), hi = min(pe, lo + per);
            int sum = 0;
            for (int p = lo; p < hi; ++p) sum += count(p);
            int inc = sum;   // inclusive prefix over the 64 lanes
            for (int d = 1; d < 64; d <<= 1) {
                const int v = __shfl_up(inc, d, 64);
                if (lane >= d) inc += v;
            }
            __builtin_amdgcn_wave_barrier();
            const int base = (int)x0 - a0;   // column of LDS byte 0
            auto put = [&](int c, int q) __attribute__((always_inline)) {   // residue q in column c
                if (c >= (int)x0 && c < x1 && q < n) buf[c - base] = rl ? sres[q] : gres[q];
            };
            int q = qa + inc - sum;
            for (int u = 0; u < per; ++u) {   // uniform trip count (ballots)
                const int p = lo + u;
                const bool act = p < hi;
                const int ni = act ? (int)sins[p] : 0;
                const int2 cg = act ? colg(p) : make_int2(0, 0);
                if (ni <= kRowFew)
                    for (int t = 0; t < ni; ++t) put(cg.x + t, q + t);
                uint64_t big = __ballot(ni > kRowFew);
                while (big) {
                    const int l = __builtin_ctzll(big);
                    big &= big - 1;
                    const int bn = __builtin_amdgcn_readlane(ni, l), bc = __builtin_amdgcn_readlane(cg.x, l),
                              bq = __builtin_amdgcn_readlane(q, l);
                    for (int t = lane; t < bn; t += 64) put(bc + t, bq + t);
                }
                q += ni;
                if (act && p < m && ((abit[p >> 5] >> (p & 31)) & 1u)) {
                    put(cg.x + cg.y, q);
                    ++q;
                }
            }
            __builtin_amdgcn_wave_barrier();
            // copy out: LDS byte a0 + c holds column x0 + c
            uint8_t *dst = row + x0 - a0;   // 16-byte aligned (x0 is a multiple of 16)
            for (int w = lane; w < nw; w += 64) {
                const int b0 = 16 * w;
                if (b0 >= a0 && b0 + 16 <= a0 + len) {
                    *reinterpret_cast<uint4 *>(dst + b0) = buf16[w];
                } else {
                    for (int c = max(b0, a0); c < min(b0 + 16, a0 + len); ++c) dst[c] = buf[c];
                }
            }
            __builtin_amdgcn_wave_barrier();
            if (x1 < width) {   // the next chunk's first block holds column x1 or starts there
                const bool whole = pe < m1 && colv(pe) == x1;
                qa += __builtin_amdgcn_readlane(inc, 63) - (whole ? 0 : count(pe - 1));
                pa = whole ? pe : pe - 1;
            }
        }
        if (!more) break;
    }
}

constexpr int kRowsChunkMinBlocks = 4096;   // centers with more blocks take the chunked row kernels
constexpr int kRowChunk = 256;              // blocks per task, four per lane
constexpr int kRowWin = 2048;               // LDS bytes of a task's column window
constexpr int kRowRes = 2048;               // LDS bytes of a task's residues (more: read from global memory)
constexpr int kRowWave = kRowWin + 16 + kRowRes + 16;   // LDS bytes per wavefront

// Chunked rows, first pass, one workgroup per row: ck[k][c] = residues of row
// k before block c * kRowChunk (insertions plus aligned bits).  A wavefront counts a
// chunk with two loads of aligned words (pairs of counts) per lane, four chunks in
// flight on each of eight wavefronts; the counts of up to kRowTile chunks (65,536
// blocks, which hold the center of any sequence; vectors made elsewhere may have more) meet
// in LDS, and the row's sum is carried from one such tile to the next.  One wavefront per row that
// carried its sum from chunk to chunk took 66 us at 672 rows of 16,570 blocks (22 MB).
constexpr int kRowTile = 256;
__global__ void __launch_bounds__(512) rows_count_kernel(RowsArgs a, int32_t *ck, int nck) {
    __shared__ int s_cnt[kRowTile], s_wave[8];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = a.m, m1 = m + 1;
    for (int k = blockIdx.x; k < a.nrows; k += gridDim.x) {
        const uint16_t *ir = a.ins + (int64_t)k * m1;
        const uint32_t *ar = a.aligned + (int64_t)k * a.aw;
        int carry = 0;   // residues before the tile
        for (int t0 = 0; t0 < nck; t0 += kRowTile) {
            const int nt = min(kRowTile, nck - t0);
            for (int c0 = wv; c0 < nt; c0 += 32) {
                int v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int b = (t0 + c0 + 8 * u) * kRowChunk, nb = min(kRowChunk, m1 - b);   // (nb <= 0: no such chunk)
                    const uintptr_t p = (uintptr_t)(ir + b);
                    const int odd = (int)((p >> 1) & 1);
                    const uint32_t *w = reinterpret_cast<const uint32_t *>(p & ~(uintptr_t)3);
                    v[u] = 0;
                    if (nb <= 0) continue;
#pragma unroll
                    for (int r = 0; r < 3; ++r) {   // word i holds the counts 2i - odd and 2i + 1 - odd
                        const int i = 64 * r + lane, lo = 2 * i - odd;
                        if (r == 2 && (lane > 0 || !odd)) continue;
                        if (lo >= nb) continue;
                        const uint32_t x = w[i];
                        v[u] += (lo >= 0 ? (int)(x & 0xffffu) : 0) + (lo + 1 < nb ? (int)(x >> 16) : 0);
                    }
                    if (lane < 8 && b + 32 * lane < m) {   // the aligned words of center positions b + 32 lane ..
                        const int left = m - (b + 32 * lane);
                        v[u] += __popc(ar[(b >> 5) + lane] & (left >= 32 ? ~0u : (1u << left) - 1u));
                    }
                }
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] += __shfl_xor(v[u], o, 64);
                if (lane < 4 && c0 + 8 * lane < nt)
                    s_cnt[c0 + 8 * lane] = lane == 0 ? v[0] : lane == 1 ? v[1] : lane == 2 ? v[2] : v[3];
            }
            __syncthreads();
            const int own = tid < nt ? s_cnt[tid] : 0;
            int inc = own;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int t = __shfl_up(inc, d, 64);
                if (lane >= d) inc += t;
            }
            if (lane == 63) s_wave[wv] = inc;
            __syncthreads();
            int before = carry + inc - own;
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                if (w < wv) before += s_wave[w];
                carry += s_wave[w];
            }
            if (tid < nt) ck[(int64_t)k * nck + t0 + tid] = before;
            __syncthreads();
        }
    }
}

// Chunked rows, second pass: one wavefront per (row k, chunk c) task, lane L
// owning blocks p = c * kRowChunk + 4L + u (u < 4).  Wave prefix sums over the
// lanes give each lane its first residue (from ck) and first column (from
// col[c * kRowChunk]); the chunk's residues are staged in LDS (coalesced), and
// its columns are built in an LDS window of kRowWin bytes at a time (filled
// with gaps, then each residue placed: block p's insertion t at its column +
// t, its aligned residue at its column + G[p]) and copied out with 16-byte
// stores, byte stores where a 16-byte word is shared with a neighbouring
// chunk.  The window sits in LDS at the
// output's misalignment, so aligned LDS words map onto aligned global words.
// A task's counts, columns and bits are loaded a task ahead: 672 rows of 16,570
// blocks and 18,611 columns take 46 us, 53 with all loads in line.
__global__ void __launch_bounds__(256) rows_chunk_kernel(RowsArgs a, const int32_t *ck, int nck) {
    extern __shared__ uint4 lds_rows[];
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint8_t *buf = reinterpret_cast<uint8_t *>(lds_rows) + wid * kRowWave;
    uint4 *buf16 = reinterpret_cast<uint4 *>(buf);
    uint8_t *rbuf = buf + kRowWin + 16;   // the task's residues
    const int m = a.m, m1 = m + 1;
    const int64_t width = a.width;
    const int64_t ntask = (int64_t)a.nrows * nck, tstep = (int64_t)gridDim.x * 4;
    // what a task reads by itself, loaded a task ahead
    struct Task {
        int c, n, qt;
        int64_t k, so, colb, cole;
        int ni[4], gg[4];
        uint32_t al;
    };
    auto load = [&](int64_t task) __attribute__((always_inline)) {
        Task t;
        t.k = task / nck;
        t.c = (int)(task - t.k * nck);
        const int b = t.c * kRowChunk, bend = min(b + kRowChunk, m1), p0 = b + 4 * lane;
        t.so = a.off[t.k];
        t.n = (int)(a.off[t.k + 1] - t.so);
        t.qt = ck[task];                        // the chunk's first residue
        t.colb = a.col[b];
        t.cole = bend < m1 ? a.col[bend] : width;
        const uint16_t *ir = a.ins + t.k * m1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            t.ni[u] = p0 + u < bend ? (int)ir[p0 + u] : 0;
            t.gg[u] = p0 + u < bend ? a.G[p0 + u] : 0;
        }
        t.al = p0 < m ? a.aligned[t.k * a.aw + (p0 >> 5)] : 0u;
        return t;
    };
    int64_t task = (int64_t)blockIdx.x * 4 + wid;
    if (task >= ntask) return;
    Task nx = load(task);
    for (; task < ntask; task += tstep) {
        const Task cur = nx;
        if (task + tstep < ntask) nx = load(task + tstep);
        const int c = cur.c, n = cur.n, qt = cur.qt;
        const int b = c * kRowChunk, bend = min(b + kRowChunk, m1);
        const uint8_t *s = a.res + cur.so;
        const int p0 = b + 4 * lane;
        const int *ni = cur.ni, *gg = cur.gg;
        const uint32_t al4 = p0 < m ? (cur.al >> (p0 & 31)) & ((1u << min(4, m - p0)) - 1u) : 0u;
        int nres = 0, ncol = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            nres += ni[u] + (int)((al4 >> u) & 1u);
            ncol += p0 + u < bend ? gg[u] + (p0 + u < m ? 1 : 0) : 0;
        }
        int ir_ = nres, ic_ = ncol;   // inclusive prefix sums over the lanes
        for (int d = 1; d < 64; d <<= 1) {
            const int t1 = __shfl_up(ir_, d, 64), t2 = __shfl_up(ic_, d, 64);
            if (lane >= d) {
                ir_ += t1;
                ic_ += t2;
            }
        }
        const int q0 = qt + ir_ - nres;         // the lane's first residue
        // the chunk's residues qt .. qt + ntot - 1 into LDS as aligned words
        // (each holds a residue of the row, so it never leaves its page), when
        // they fit
        const int ntot = __shfl(ir_, 63, 64);
        const bool rl = ntot <= kRowRes;
        const uintptr_t sa = (uintptr_t)(s + qt);
        const int ro = (int)(sa & 3), nb = min(ntot, n - qt), nwd = rl && nb > 0 ? (ro + nb + 3) >> 2 : 0;
        const uint32_t *sw = reinterpret_cast<const uint32_t *>(sa & ~(uintptr_t)3);
        uint32_t *rw = reinterpret_cast<uint32_t *>(rbuf);
        for (int i0 = 0; i0 < nwd; i0 += 256) {
            uint32_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = i0 + 64 * u + lane < nwd ? sw[i0 + 64 * u + lane] : 0u;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i0 + 64 * u + lane < nwd) rw[i0 + 64 * u + lane] = v[u];
        }
        auto resid = [&](int r) __attribute__((always_inline)) -> uint8_t {
            return r >= n ? (uint8_t)255 : (rl ? rbuf[r - qt + ro] : s[r]);
        };
        const int64_t colb = cur.colb, span = cur.cole - colb;
        const int cl = ic_ - ncol;              // the lane's first column, relative to colb
        uint8_t *row = a.msa + cur.k * width;
        const int a0 = (int)((uintptr_t)(row + colb) & 15);
        for (int64_t x0 = 0; x0 < span; x0 += kRowWin) {
            const int wl = (int)min<int64_t>(kRowWin, span - x0);
            const int nw = (a0 + wl + 15) >> 4;
            for (int q = lane; q < nw; q += 64) buf16[q] = make_uint4(~0u, ~0u, ~0u, ~0u);
            __builtin_amdgcn_wave_barrier();
            int cu = cl, qu = q0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (p0 + u < bend) {
                    // insertions t at cu + t, for the t inside the window
                    const int64_t t0 = max<int64_t>(0, x0 - cu), t1 = min<int64_t>(ni[u], x0 + wl - cu);
                    for (int64_t t = t0; t < t1; ++t) buf[a0 + (int)(cu + t - x0)] = resid(qu + (int)t);
                    qu += ni[u];
                    if (p0 + u < m) {
                        if ((al4 >> u) & 1u) {
                            const int64_t pos = (int64_t)cu + gg[u] - x0;
                            if (pos >= 0 && pos < wl) buf[a0 + (int)pos] = resid(qu);
                            ++qu;
                        }
                        cu += gg[u] + 1;
                    } else {
                        cu += gg[u];
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
            uint8_t *dst = row + colb + x0 - a0;   // 16-byte aligned
            for (int q = lane; q < nw; q += 64) {
                const int b0 = 16 * q;
                if (b0 >= a0 && b0 + 16 <= a0 + wl) {
                    *reinterpret_cast<uint4 *>(dst + b0) = buf16[q];
                } else {
                    for (int e = max(b0, a0); e < min(b0 + 16, a0 + wl); ++e) dst[e] = buf[e];
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

constexpr int kProfCols = 256;      // columns per workgroup (four per lane)
constexpr int kProfMaxSlab = 65535; // rows per workgroup (16-bit partial counts)
constexpr int kProfRows = 16;       // rows loaded per pass of a wavefront

// Column profile of an N x W MSA, first pass: workgroup (x, y) counts the
// bytes of columns 256 x .. 256 x + 255 over the rows of slab y, its four
// wavefronts taking rows in turn.  A lane loads four columns at once (a
// wavefront 256 consecutive bytes of a row, at any alignment), 16 rows before
// they are counted.  With a byte per lane the loads' issue bounded the kernel
// (1e6 x 1,000: 234 us with the counting alone
// against 163).  The counters sit in LDS:
// word bin * 256 + 64 (column % 4) + column / 4, so the lanes of one count are on
// distinct banks; bin 0 counts gaps, bin 1 + a residue code a, bin alpha + 1 any
// other byte (which raises *bad).  The slab's counts go, without atomics, to
// part[y][column][slot] (uint16; slot a < alpha a residue code, slot alpha the
// gaps), written in contiguous runs.  EDGE: the last columns of an MSA at least
// four wide; a lane with fewer than four (cols) loads the row's last four bytes
// and shifts, and what lies past the end counts into a bin that is discarded.
template <bool EDGE>
__device__ __forceinline__ void colprof_rows(const uint8_t *p, int64_t step, int rows, int cols, uint32_t *lc,
                                             uint32_t top) {
    const int sh = EDGE ? 8 * (4 - cols) & 31 : 0;
    auto load = [&](const uint8_t *q) __attribute__((always_inline)) {
        uint32_t v;
        __builtin_memcpy(&v, q, 4);
        return EDGE ? v >> sh : v;
    };
    auto count = [&](uint32_t v) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t bin = min((((v >> (8 * k)) & 255u) + 1u) & 255u, top);
            if (EDGE && k >= cols) bin = top + 1u;
            atomicAdd(lc + bin * 256 + 64 * k, 1u);
        }
    };
    int r = 0;
    for (; r + kProfRows <= rows; r += kProfRows, p += kProfRows * step) {
        uint32_t v[kProfRows];
#pragma unroll
        for (int u = 0; u < kProfRows; ++u) v[u] = load(p + u * step);
#pragma unroll
        for (int u = 0; u < kProfRows; ++u) count(v[u]);
    }
    for (; r < rows; ++r, p += step) count(load(p));
}

__global__ void __launch_bounds__(256)
colprof_kernel(const uint8_t *msa, int n, int64_t width, int alpha, int slab, uint16_t *part, uint32_t *bad, uint32_t tag) {
    extern __shared__ uint32_t pcnt[];
    const int nbin = alpha + 3;
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    for (int x = t; x < nbin * 256; x += 256) pcnt[x] = 0;
    __syncthreads();
    const int64_t cb = (int64_t)blockIdx.x * kProfCols;
    const int r0 = blockIdx.y * slab;
    const int r1 = min(n, r0 + slab);
    const int cols = (int)min((int64_t)4, max((int64_t)0, width - (cb + 4 * lane)));   // this lane's columns
    const uint8_t *p = msa + (int64_t)(r0 + wave) * width + cb + 4 * lane;
    const int rows = (r1 - r0 - wave + 3) >> 2;   // rows r0 + wave, + 4, ...
    const uint32_t top = (uint32_t)alpha + 1u;
    if (cb + kProfCols <= width) {
        colprof_rows<false>(p, 4 * width, rows, 4, pcnt + lane, top);
    } else if (width >= 4) {   // lanes past the end read the last four columns too
        colprof_rows<true>(msa + (int64_t)(r0 + wave) * width + min(cb + 4 * lane, width - 4), 4 * width, rows, cols,
                           pcnt + lane, top);
    } else if (cols > 0) {
        for (int r = 0; r < rows; ++r, p += 4 * width)
            for (int k = 0; k < cols; ++k) atomicAdd(pcnt + min((p[k] + 1u) & 255u, top) * 256 + 64 * k + lane, 1u);
    }
    __syncthreads();
    if (pcnt[top * 256 + t] != 0) atomicMax(bad, tag);
    // slab counts out: element e of the workgroup's run is (column e / nsym, slot e % nsym)
    const int nsym = alpha + 1;
    const int64_t ncols = min((int64_t)kProfCols, width - cb);
    uint16_t *dst = part + ((int64_t)blockIdx.y * width + cb) * nsym;
    for (int e = t; e < ncols * nsym; e += 256) {
        const int c = e / nsym, slot = e - c * nsym;
        dst[e] = (uint16_t)pcnt[(slot == alpha ? 0 : slot + 1) * 256 + 64 * (c & 3) + (c >> 2)];
    }
}

// element e of the profile: its slabs' counts added, eight loads in flight
__device__ __forceinline__ int32_t colprof_total(const uint16_t *part, int nslab, int64_t nelem, int64_t e) {
    int32_t s = 0;
#pragma unroll 8
    for (int y = 0; y < nslab; ++y) s += part[(int64_t)y * nelem + e];
    return s;
}

// Second pass: profile[e] = sum over slabs of part[slab][e], e < width * nsym.
__global__ void __launch_bounds__(256)
colprof_sum_kernel(const uint16_t *part, int nslab, int64_t nelem, int32_t *prof) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e < nelem) prof[e] = colprof_total(part, nslab, nelem, e);
}

struct SpMatrix {
    int8_t s[kAlphaMax * kAlphaMax];   // alpha x alpha
};

// avg SP numerator and BLOSUM column SP from the slabs' counts, summed over the
// workgroup's columns into out[2 * workgroup] += (pairs of different residues) +
// 2 * (residue-gap pairs) and out[.. + 1] += sum of S over residue pairs - ge *
// (residue-gap pairs).  A workgroup totals eight columns at a time into LDS,
// then its threads share the columns' residue pairs (with a thread per column
// the 16 workgroups of 4,030 columns took 23 us, after a 20 us pass that wrote
// the profile; now 15).
constexpr int kSpCols = 8, kSpGroups = 512;   // columns at a time, workgroups at most
__global__ void __launch_bounds__(256)
sp_profile_kernel(const uint16_t *part, int nslab, int64_t width, int alpha, SpMatrix mat, int ge, int64_t *out) {
    __shared__ int32_t cnt[kSpCols * (kAlphaMax + 1)];
    __shared__ int8_t smat[kAlphaMax * kAlphaMax];
    __shared__ long long red[2][4];
    const int tid = threadIdx.x, nsym = alpha + 1;
    for (int x = tid; x < alpha * alpha; x += 256) smat[x] = mat.s[x];
    long long sp = 0, bl = 0;
    for (int64_t c0 = (int64_t)blockIdx.x * kSpCols; c0 < width; c0 += (int64_t)gridDim.x * kSpCols) {
        const int nc = (int)min((int64_t)kSpCols, width - c0);
        __syncthreads();   // the previous columns' counts are done with
        for (int e = tid; e < nc * nsym; e += 256)
            cnt[e] = colprof_total(part, nslab, width * nsym, c0 * nsym + e);
        __syncthreads();
        // item (column, a): residue a against itself and every later code
        for (int q = tid; q < nc * alpha; q += 256) {
            const int32_t *c = cnt + q / alpha * nsym;
            const int a = q % alpha;
            const int64_t ca = c[a], g = c[alpha];
            if (!ca) continue;
            int64_t later = 0;
            bl += ca * (ca - 1) / 2 * smat[a * alpha + a] - (int64_t)ge * g * ca;
            for (int b = a + 1; b < alpha; ++b) {
                later += c[b];
                bl += ca * (int64_t)c[b] * smat[a * alpha + b];
            }
            sp += ca * later + 2 * g * ca;
        }
    }
    for (int d = 32; d > 0; d >>= 1) {
        sp += __shfl_xor(sp, d);
        bl += __shfl_xor(bl, d);
    }
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = sp;
        red[1][tid >> 6] = bl;
    }
    __syncthreads();
    if (tid < 2) out[2 * blockIdx.x + tid] = red[tid][0] + red[tid][1] + red[tid][2] + red[tid][3];
}

}  // namespace hk

// Small kernels around the wavefront forward pass: staging of stream
// residues and decoding of the end-cell keys.
#pragma once
#include "sw_kernels.hpp"

namespace hk {

// keys -> score and end cell (i1, j1), 1-based, and the score-only cells (0, 0,
// i1, j1); slot q belongs to pair pid[q].
__global__ void decode_keys_kernel(const unsigned long long *keys, const int32_t *slot_pid, int nslots,
                                   int32_t *score, int32_t *endcell, int4 *cells) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nslots) return;
    const unsigned long long k = keys[q];
    const int pid = slot_pid[q];
    const int h = (int)(k >> 32);
    score[pid] = h;
    const int i1 = h > 0 ? 0xffff - (int)(k & 0xffff) + 1 : 0, j1 = h > 0 ? 0xffff - (int)((k >> 16) & 0xffff) : 0;
    if (endcell) {
        endcell[2 * pid] = i1;
        endcell[2 * pid + 1] = j1;
    }
    if (cells) cells[pid] = make_int4(0, 0, i1, j1);
}

// Stage the residues of every stream: sres[sbase + c0(q) + x] = s_q[x], with
// kFirstCol on x = 0, and clear the slot's end-cell key.  One workgroup per
// pair slot.
__global__ void stage_stream_kernel(const uint8_t *res, const int64_t *off, const int32_t *slot_pid,
                                    const int64_t *slot_col, int nslots, int clamp, uint8_t *sres,
                                    unsigned long long *keys) {
    const int q = blockIdx.x;
    if (q >= nslots) return;
    if (threadIdx.x == 0) keys[q] = 0ull;
    const int pid = slot_pid[q];
    const int64_t so = off[pid];
    const int n = (int)(off[pid + 1] - so);
    uint8_t *dst = sres + slot_col[q];
    for (int x = threadIdx.x; x < n; x += blockDim.x)
        dst[x] = (uint8_t)(min((int)(res[so + x] & 31), clamp) | (x == 0 ? kFirstCol : 0));
}

// ---- streams planned on the device ---------------------------------------------
// The host's counting sort, dealing and slot arrays take about 140 us at 20,000
// pairs and 1.6 ms at 300,000, during which the device waits.  Here the pairs are
// sorted by length (three small kernels) and dealt by formula: the x-th longest, x =
// r * ns + j, goes to stream j in even rounds r and ns - 1 - j in odd ones, so
// two streams differ by at most the longest pair, and every stream gets a region
// of the same size for its columns, codes and boundary rows, bounded by the
// average load plus the longest pair.
struct DevPlanArgs {
    const uint8_t *res;
    const int64_t *off;
    int np, maxlen, ns, clamp;   // ns <= np
    int32_t *hist;        // [maxlen + 1], zeroed; then each length's next place
    int2 *order;          // [np] (pair, length), longest first
    int per_group;        // streams that share codes and boundary rows (2: packed)
    int64_t cols, code_words, bound_elems;   // region sizes: columns per stream, the others per group
    int32_t *spid, *sstr, *slot0, *slen;
    int64_t *scol, *sbeg, *scb, *sbb;
    unsigned long long *keys;
    uint8_t *sres;
};
constexpr int kPlanHistLds = 8192;   // lengths counted in LDS first

__global__ void __launch_bounds__(256) plan_hist_kernel(DevPlanArgs a) {
    __shared__ int32_t h[kPlanHistLds];
    const bool lds = a.maxlen < kPlanHistLds;
    if (lds) {
        for (int x = threadIdx.x; x <= a.maxlen; x += 256) h[x] = 0;
        __syncthreads();
    }
    for (int x = blockIdx.x * 256 + threadIdx.x; x < a.np; x += gridDim.x * 256)
        atomicAdd((lds ? h : a.hist) + (int)(a.off[x + 1] - a.off[x]), 1);
    if (!lds) return;
    __syncthreads();
    for (int x = threadIdx.x; x <= a.maxlen; x += 256)
        if (h[x]) atomicAdd(a.hist + x, h[x]);
}

// hist[L] -> pairs longer than L, one workgroup
__global__ void __launch_bounds__(1024) plan_scan_kernel(int32_t *hist, int maxlen) {
    __shared__ int32_t part[1024];
    const int tid = threadIdx.x, n = maxlen + 1, per = (n + 1023) / 1024;
    const int lo = min(n, tid * per), hi = min(n, lo + per);   // positions in descending length
    int sum = 0;
    for (int p = lo; p < hi; ++p) sum += hist[maxlen - p];
    part[tid] = sum;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int v = tid >= d ? part[tid - d] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int acc = tid > 0 ? part[tid - 1] : 0;
    for (int p = lo; p < hi; ++p) {
        const int c = hist[maxlen - p];
        hist[maxlen - p] = acc;
        acc += c;
    }
}

__global__ void __launch_bounds__(256) plan_scatter_kernel(DevPlanArgs a) {
    const int x = blockIdx.x * 256 + threadIdx.x;
    if (x >= a.np) return;
    const int L = (int)(a.off[x + 1] - a.off[x]);
    a.order[atomicAdd(a.hist + L, 1)] = make_int2(x, L);
}

// One wavefront per pair in length order: its slot, its stream column, its
// residues staged as stage_stream_kernel does; the first round's wavefronts also
// write their stream's entries.
__global__ void __launch_bounds__(256) plan_stage_kernel(DevPlanArgs a) {
    const int x = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (x >= a.np) return;
    const int ns = a.ns, r = x / ns, j = x - r * ns;
    const int s = (r & 1) ? ns - 1 - j : j;
    const int rounds = a.np / ns, rem = a.np - rounds * ns;   // full rounds, pairs of the last one
    // pairs of the streams before s in the last round, and whether s has one
    const int before = (rounds & 1) ? max(0, s - (ns - rem)) : min(s, rem);
    const bool last = (rounds & 1) ? s >= ns - rem : s < rem;
    const int first = s * rounds + before;
    const int upto = r == 0 ? rounds + (last ? 1 : 0) : r;   // all pairs of the stream, or the earlier ones
    const int2 pl = a.order[x];
    int64_t c = 0;
    for (int q = lane; q < upto; q += 64) c += a.order[(int64_t)q * ns + ((q & 1) ? ns - 1 - s : s)].y;
    for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d);
    const int64_t base = (int64_t)s * a.cols;
    if (r == 0) {
        if (lane == 0) {
            a.sbeg[s] = base;
            a.slen[s] = (int32_t)c;
            a.slot0[s] = first;
            a.scb[s] = s / a.per_group * a.code_words;
            a.sbb[s] = s / a.per_group * a.bound_elems;
        }
        c = 0;
    }
    if (lane == 0) {
        const int q = first + r;
        a.spid[q] = pl.x;
        a.scol[q] = base + c;
        a.sstr[q] = s;
        a.keys[q] = 0ull;
    }
    const uint8_t *src = a.res + a.off[pl.x];
    uint8_t *dst = a.sres + base + c;
    for (int y = lane; y < pl.y; y += 64)
        dst[y] = (uint8_t)(min((int)(src[y] & 31), a.clamp) | (y == 0 ? kFirstCol : 0));
}

}  // namespace hk

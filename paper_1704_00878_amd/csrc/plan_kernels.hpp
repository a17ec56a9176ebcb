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

// The n residues at src into dst by a wavefront, each code & 31 and at most
// clamp (<= 31), with kFirstCol on the first one: aligned words of dst, each put
// together from two aligned words of src (a word that holds a residue never leaves
// its page), and single bytes at both ends, whose words other pairs share.  A byte
// per lane took 220 us for 300,000 pairs (157 MB).
__device__ __forceinline__ void stage_pair(const uint8_t *src, int n, uint8_t *dst, int clamp, int lane) {
    const int head = min(n, (int)((4 - ((uintptr_t)dst & 3)) & 3)), nw = (n - head) >> 2, tail = n - head - 4 * nw;
    const uint32_t c4 = (uint32_t)clamp * 0x01010101u;
    const uintptr_t sa = (uintptr_t)(src + head);
    const uint32_t *sw = reinterpret_cast<const uint32_t *>(sa & ~(uintptr_t)3);
    const int sh = 8 * (int)(sa & 3);
    uint32_t *dw = reinterpret_cast<uint32_t *>(dst + head);
    for (int i = lane; i < nw; i += 64) {
        const uint32_t w0 = sw[i], w1 = sh ? sw[i + 1] : 0u;
        const uint32_t x = (uint32_t)(((uint64_t)w1 << 32 | w0) >> sh) & 0x1f1f1f1fu;
        const uint32_t over = ((((x | 0x80808080u) - c4) & 0x80808080u) >> 7) * 255u;   // bytes >= clamp
        const uint32_t y = (x & ~over) | (c4 & over);
        dw[i] = y | (i == 0 && head == 0 ? (uint32_t)kFirstCol : 0u);
    }
    const int e = lane < head ? lane : n - tail + lane - 8;   // lanes 0 .. 2: the head, 8 .. 10: the tail
    if (lane < head || (lane >= 8 && lane < 8 + tail))
        dst[e] = (uint8_t)(min((int)(src[e] & 31), clamp) | (e == 0 ? kFirstCol : 0));
}

// Stage the residues of every stream: sres[c(q) + x] = s_q[x], and clear the
// slot's end-cell key.  One wavefront per pair slot.  A small plan is read from
// pinned host memory, and further workgroups copy it to the device (psrc, n16
// 16-byte words) for the kernels after this one: a copy of its own cost 8 us.
__global__ void __launch_bounds__(256) stage_stream_kernel(const uint8_t *res, const int64_t *off,
                                                           const int32_t *slot_pid, const int64_t *slot_col, int nslots,
                                                           int clamp, uint8_t *sres, unsigned long long *keys,
                                                           const uint4 *psrc, uint4 *pdst, int n16) {
    const int wgs = (nslots + 3) / 4;
    if ((int)blockIdx.x >= wgs) {
        const int x = ((int)blockIdx.x - wgs) * 256 + threadIdx.x;
        if (x < n16) pdst[x] = psrc[x];
        return;
    }
    const int q = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (q >= nslots) return;
    if (lane == 0) keys[q] = 0ull;
    const int pid = slot_pid[q];
    const int64_t so = off[pid];
    stage_pair(res + so, (int)(off[pid + 1] - so), sres + slot_col[q], clamp, lane);
}

// ---- streams planned on the device ---------------------------------------------
// The host's counting sort, dealing and slot arrays take about 140 us at 20,000
// pairs and 1.6 ms at 300,000, during which the device waits.  Here the pairs are
// sorted by length (three small kernels) and dealt by formula: the `own` longest to
// a stream each, and of the rest the x-th longest, x = r * (ns - own) + j, to the
// j-th other stream in even rounds r and to the j-th from the end in odd ones.  Two of
// those streams differ by at most their longest pair, and every stream gets a
// region of the same size for its columns, codes and boundary rows, bounded by
// the average of all pairs over ns - own streams plus the longest pair.
struct DevPlanArgs {
    const uint8_t *res;
    const int64_t *off;
    int np, maxlen, ns, own, clamp;   // own < ns <= np
    int32_t *hist;        // [maxlen + 1]: each length's next place
    int2 *order;          // [np] (pair, length), longest first
    int per_group;        // streams that share codes and boundary rows (2: packed)
    int64_t cols, code_words, bound_elems;   // region sizes: columns per stream, the others per group
    int32_t *spid, *sstr, *slot0, *slen;
    int64_t *scol, *sbeg, *scb, *sbb;
    unsigned long long *keys;
    uint8_t *sres;
};
constexpr int kPlanHistLds = 8192;   // lengths counted in LDS

// Counts into zeroed hist, where the call's first kernel has not counted (from
// lengths of kPrepHistMax on).
__global__ void __launch_bounds__(256) plan_hist_kernel(DevPlanArgs a) {
    for (int x = blockIdx.x * 256 + threadIdx.x; x < a.np; x += gridDim.x * 256)
        atomicAdd(a.hist + (int)(a.off[x + 1] - a.off[x]), 1);
}

// hist[L] -> pairs longer than L, one workgroup; part (optional): nparts rows
// of counts to add up instead
__global__ void __launch_bounds__(1024) plan_scan_kernel(int32_t *hist, int maxlen, const int32_t *part, int nparts) {
    __shared__ int32_t psum[1024];
    const int tid = threadIdx.x, n = maxlen + 1, per = (n + 1023) / 1024;
    const int lo = min(n, tid * per), hi = min(n, lo + per);   // positions in descending length
    int sum = 0;
    for (int p = lo; p < hi; ++p) {
        const int L = maxlen - p;
        if (part) {
            int c = 0;
#pragma unroll 8
            for (int b = 0; b < nparts; ++b) c += part[b * n + L];
            hist[L] = c;
            sum += c;
        } else {
            sum += hist[L];
        }
    }
    psum[tid] = sum;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int v = tid >= d ? psum[tid - d] : 0;
        __syncthreads();
        psum[tid] += v;
        __syncthreads();
    }
    int acc = tid > 0 ? psum[tid - 1] : 0;
    for (int p = lo; p < hi; ++p) {
        const int c = hist[maxlen - p];
        hist[maxlen - p] = acc;
        acc += c;
    }
}

// Pairs to their places in length order.  A workgroup ranks its pairs within
// each length in LDS and takes a length's places with one atomic (an atomic per
// pair on its length took 66 us at 300,000 pairs of 1,000 lengths).
constexpr int kScatterPer = 2;
__global__ void __launch_bounds__(1024) plan_scatter_kernel(DevPlanArgs a) {
    __shared__ int32_t h[kPlanHistLds];
    const int tid = threadIdx.x;
    const bool lds = a.maxlen < kPlanHistLds;
    int len[kScatterPer], at[kScatterPer];
    if (lds) {
        for (int x = tid; x <= a.maxlen; x += 1024) h[x] = 0;
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kScatterPer; ++u) {
        const int x = (blockIdx.x * kScatterPer + u) * 1024 + tid;
        len[u] = x < a.np ? (int)(a.off[x + 1] - a.off[x]) : -1;
        at[u] = len[u] >= 0 ? atomicAdd((lds ? h : a.hist) + len[u], 1) : 0;
    }
    if (lds) {
        __syncthreads();
        for (int x = tid; x <= a.maxlen; x += 1024) {
            const int c = h[x];
            if (c) h[x] = atomicAdd(a.hist + x, c);
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kScatterPer; ++u)
        if (len[u] >= 0)
            a.order[at[u] + (lds ? h[len[u]] : 0)] = make_int2((blockIdx.x * kScatterPer + u) * 1024 + tid, len[u]);
}

// One wavefront per pair in length order: its slot, its stream column, its
// residues staged; the first round's wavefronts also
// write their stream's entries.
__global__ void __launch_bounds__(256) plan_stage_kernel(DevPlanArgs a) {
    const int x = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (x >= a.np) return;
    const bool own = x < a.own;   // (the only pair of stream x)
    const int ns = a.ns - a.own, np = a.np - a.own;   // the dealt pairs and their streams
    const int xd = x - a.own, r = own ? 0 : xd / ns, j = xd - r * ns;
    const int s = (r & 1) ? ns - 1 - j : j;
    const int rounds = np / ns, rem = np - rounds * ns;   // full rounds, pairs of the last one
    // pairs of the streams before s in the last round, and whether s has one
    const int before = (rounds & 1) ? max(0, s - (ns - rem)) : min(s, rem);
    const bool last = (rounds & 1) ? s >= ns - rem : s < rem;
    const int first = own ? x : a.own + s * rounds + before, sg = own ? x : a.own + s;   // first slot, stream of all
    const int upto = r == 0 ? rounds + (last ? 1 : 0) : r;   // all pairs of the stream, or the earlier ones
    const int2 pl = a.order[x];
    int64_t c = 0;
    if (own) {
        c = pl.y;
    } else {
        for (int q = lane; q < upto; q += 64) c += a.order[a.own + (int64_t)q * ns + ((q & 1) ? ns - 1 - s : s)].y;
        for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d);
    }
    const int64_t base = (int64_t)sg * a.cols;
    if (r == 0) {
        if (lane == 0) {
            a.sbeg[sg] = base;
            a.slen[sg] = (int32_t)c;
            a.slot0[sg] = first;
            a.scb[sg] = sg / a.per_group * a.code_words;
            a.sbb[sg] = sg / a.per_group * a.bound_elems;
        }
        c = 0;
    }
    if (lane == 0) {
        const int q = first + r;
        a.spid[q] = pl.x;
        a.scol[q] = base + c;
        a.sstr[q] = sg;
        a.keys[q] = 0ull;
    }
    stage_pair(a.res + a.off[pl.x], pl.y, a.sres + base + c, a.clamp, lane);
}

}  // namespace hk

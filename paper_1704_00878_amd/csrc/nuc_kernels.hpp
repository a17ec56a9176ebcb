// Nucleotide center star for gfx950 (Methods, trie section): the center's
// segments of k bases are indexed, each sequence is scanned for them, the
// largest co-linear chain of non-overlapping matches becomes its anchors, and
// only the stretches between anchors are aligned (end to end, affine gaps).
//
// The paper indexes the segments in a trie with failure links, which reports
// every occurrence of every segment in one left-to-right pass.  Here the same
// set of occurrences comes from a hash table of the segments' 2-bit packed
// strings (one probe per position of the sequence); the table is built on the
// device and sits in LDS.
//
// Four kernels, each bound by latency rather than by bytes (672 genomes of
// 16,569 bases: 11 MB in, 22 MB of insertion counts): the table by one workgroup, the
// scan by a wavefront per run of 256 match starts, the chain by a workgroup per
// sequence, which also settles the stretches that need no dynamic program,
// and the remaining stretches by a wavefront each.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hk {

constexpr int kNucNeg = -(1 << 29);

struct NucArgs {
    const uint8_t *res;       // residue codes (0..3 = A C G T, 4 = other)
    const int64_t *off;       // [N + 1]
    int nseq;
    const uint8_t *center;    // the center's codes
    int m, k;
    // segment table: T slots (power of two), key (2-bit packed string, base
    // t at bits 2t and 2t + 1) and segment index (-1 = empty); segscore[q] =
    // sum of S over segment q
    const unsigned long long *tkey;
    const int32_t *tseg;
    int lg_t;
    const int32_t *segscore;
    const int8_t *mat;        // alpha x alpha scores
    int alpha, go, ge;
    // scan chunks: sequence x owns chunks cbase[x] .. cbase[x+1]-1, chunk c of
    // x holding the match starts p in [c * kNucChunk, (c + 1) * kNucChunk)
    const int64_t *cbase;     // [N + 1]
    int64_t nchunk;
    int wparts;               // wavefronts that share a sequence's chunks in the scan
    int32_t *ccount;          // [nchunk] matches per chunk
    uint32_t *cmatch;         // matches in order of p: q << 8 | p within the chunk; those of chunk c of sequence x
                              // from off[x] + c * kNucChunk on (a place for every match start)
    int32_t *score;           // [N]
    uint16_t *ins;            // [N][m + 1] (zeroed)
    uint32_t *aligned;        // [N][aw] (zeroed)
    int aw;
    int32_t *G;               // optional merge: max of ins over the sequences
    int gskip;                // sequence kept out of G
    int own_row;              // its row is the gapped center: no insertions, every position aligned (else what it aligns to)
    int chain_cap;            // matches per sequence chained in LDS (<= kChainLdsMax)
    // sequences with more: five arrays of bigcap entries
    int32_t *big;
    int64_t bigcap;
    // stretches for the dynamic program: those at most kNucTinyW x kNucTinyW
    // from the front of the narrow list, other narrow ones from its back, wide
    // ones in their own; center start, center length, sequence start, its
    // length; the sequence; offsets of its boundary entries (wide) and codes
    int4 *nd, *wd;
    int32_t *nx, *wx;
    longlong2 *no, *wo;
    int64_t listcap;
    int2 *rows;
    uint32_t *codes;
    int64_t rowcap, codecap;
    int64_t lane_min;         // narrow stretches from which they take a lane each
    // zeroed before the chain kernel: boundary entries, code words, narrow
    // stretches (front | back << 32), wide ones, matches of big sequences, the
    // workgroups done.  Where one exceeds its capacity the call grows the
    // buffers and runs the chain and the stretches again.
    unsigned long long *count;
    const uint32_t *flag;     // the code check's word, for the mailbox
    int64_t *mail;            // optional: counts and flag for the host, then seq
    int64_t seq;
};
// (each counter on a cache line of its own: every sequence adds to it)
enum { kNucRows = 0, kNucCodes = 32, kNucNarrow = 64, kNucWide = 96, kNucBig = 128, kNucDone = 160, kNucCounts = 192 };

__device__ __forceinline__ bool nuc_overflow(const NucArgs &a, unsigned long long rows, unsigned long long codes,
                                             unsigned long long narrow, unsigned long long wide,
                                             unsigned long long big) {
    return rows > (unsigned long long)a.rowcap || codes > (unsigned long long)a.codecap ||
           (narrow & 0xffffffffull) + (narrow >> 32) > (unsigned long long)a.listcap ||
           wide > (unsigned long long)a.listcap || big > (unsigned long long)a.bigcap;
}

constexpr int kNucChunk = 256;   // match starts per scan chunk
constexpr int kNucKey32 = 16;    // segments up to this long: 32-bit keys in the table (scan of 672 x 16,569 46.4 us against 48.3)
constexpr int kNucSmallW = 32;   // stretches at most this many columns wide: one lane, the row in registers
constexpr int kNucTinyW = 20;    // narrow stretches at most this size both ways are listed apart
constexpr int kNucTallH = 40;    // stretches taller than this take a wavefront too (rows across lanes)
constexpr int kNucDiagMax = 128; // stretches up to this long are tested for the plain diagonal by one lane

// The table's hash of a packed segment.
__device__ __forceinline__ uint32_t nuc_hash(unsigned long long key, int lg_t) {
    const uint32_t h = (uint32_t)key ^ (uint32_t)(key >> 32) * 0x85EBCA6Bu;
    return (h * 0x9E3779B1u) >> (32 - lg_t);
}

// segment q whose packed string is key, or a negative number (several
// segments with that string: -2); K: 32 bits where strings fit (k <= 16)
template <typename K>
__device__ __forceinline__ int nuc_lookup(const K *tk, const int32_t *ts, int lg_t, K key) {
    const uint32_t mask = (1u << lg_t) - 1u;
    uint32_t h = nuc_hash(key, lg_t);
    for (;;) {
        const int q = ts[h];
        if (q == -1) return -1;
        if (tk[h] == key) return q;
        h = (h + 1) & mask;
    }
}

// Table in LDS when it fits (32 or 48 KiB), else read from global memory.
constexpr int kNucLdsSlots = 4096;

// Keys of type K (a.tkey holds 32-bit ones where k <= 16).
#define NUC_TABLE_SETUP(K)                                                               \
    __shared__ K s_tk[kNucLdsSlots];                                                     \
    __shared__ int32_t s_ts[kNucLdsSlots];                                               \
    const int T = 1 << a.lg_t;                                                           \
    const bool tl = T <= kNucLdsSlots;                                                   \
    const K *gk = reinterpret_cast<const K *>(a.tkey);                                   \
    if (tl)                                                                              \
        for (int x = threadIdx.x; x < T; x += blockDim.x) {                              \
            s_tk[x] = gk[x];                                                             \
            s_ts[x] = a.tseg[x];                                                         \
        }                                                                                \
    __syncthreads();                                                                     \
    const K *tk = tl ? s_tk : gk;                                                        \
    const int32_t *ts = tl ? s_ts : a.tseg;

// Workgroup 0: the segment table.  Each segment's string, cleanness (codes 0..3
// only) and score from the center staged in LDS; then every clean segment claims the
// first free slot of its probe sequence, or finds an equal string there and
// marks its owner as repeated; then the owners' strings, -2 for repeated ones
// (which the paper's index leaves out).  Workgroup 1: the first scan chunk of each
// sequence.  On the host this took 190 us with its copies at 1,035 segments.
struct NucSetup {
    const uint8_t *center;
    int m, k, nsg, alpha, lg_t;
    const int8_t *mat;
    unsigned long long *tkey, *segkey;   // [T], [nsg]
    int32_t *tseg, *segscore, *segstate; // [T], [nsg], [nsg]: 0 clean, 1 repeated, 2 not clean
    const int64_t *off;
    int nseq;
    int64_t *cbase;
};
__global__ void __launch_bounds__(1024) nuc_setup_kernel(NucSetup a) {
    __shared__ uint8_t s_cen[1024 * 32];   // the bytes of 1,024 segments (workgroup 0)
    __shared__ int64_t part[1024];
    __shared__ int s_self[32];
    const int tid = threadIdx.x;
    if (blockIdx.x == 1) {
        const int n = a.nseq, per = (n + 1023) / 1024;
        const int lo = min(n, tid * per), hi = min(n, lo + per);
        auto chunks = [&](int x) __attribute__((always_inline)) -> int64_t {
            const int64_t w = a.off[x + 1] - a.off[x] - a.k + 1;
            return w > 0 ? (w + kNucChunk - 1) / kNucChunk : 0;
        };
        int64_t sum = 0;
        for (int x = lo; x < hi; ++x) sum += chunks(x);
        part[tid] = sum;
        __syncthreads();
        for (int d = 1; d < 1024; d <<= 1) {
            const int64_t v = tid >= d ? part[tid - d] : 0;
            __syncthreads();
            part[tid] += v;
            __syncthreads();
        }
        int64_t acc = part[tid] - sum;
        for (int x = lo; x < hi; ++x) {
            a.cbase[x] = acc;
            acc += chunks(x);
        }
        if (tid == 1023) a.cbase[n] = acc;
        return;
    }
    const int T = 1 << a.lg_t, k = a.k;
    for (int h = tid; h < T; h += 1024) __hip_atomic_store(a.tseg + h, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid < 32) s_self[tid] = tid < a.alpha ? a.mat[tid * a.alpha + tid] : 0;
    for (int q0 = 0; q0 < a.nsg; q0 += 1024) {
        const int nq = min(1024, a.nsg - q0);
        __syncthreads();
        for (int x = tid; x < nq * k; x += 1024) s_cen[x] = a.center[q0 * k + x];
        __syncthreads();
        if (tid < nq) {
            unsigned long long key = 0;
            int state = 0, score = 0;
            for (int t = 0; t < k; ++t) {
                const int b = s_cen[tid * k + t];
                if (b > 3) state = 2;
                key |= (unsigned long long)(b & 3) << (2 * t);
                score += s_self[b & 31];
            }
            a.segkey[q0 + tid] = key;
            a.segscore[q0 + tid] = score;
            __hip_atomic_store(a.segstate + q0 + tid, state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __threadfence_block();
    __syncthreads();
    for (int q = tid; q < a.nsg; q += 1024) {
        if (__hip_atomic_load(a.segstate + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 2) continue;
        const unsigned long long key = a.segkey[q];
        uint32_t h = nuc_hash(key, a.lg_t);
        for (;;) {   // ends: the table has twice as many slots as there are different strings
            const int old = atomicCAS(a.tseg + h, -1, q);
            if (old == -1) break;
            if (a.segkey[old] == key) {
                __hip_atomic_store(a.segstate + old, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            h = (h + 1) & (uint32_t)(T - 1);
        }
    }
    __threadfence_block();
    __syncthreads();
    for (int h = tid; h < T; h += 1024) {
        const int q = __hip_atomic_load(a.tseg + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (q < 0) continue;
        if (k <= kNucKey32) reinterpret_cast<uint32_t *>(a.tkey)[h] = (uint32_t)a.segkey[q];
        else a.tkey[h] = a.segkey[q];
        if (__hip_atomic_load(a.segstate + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 1) a.tseg[h] = -2;
    }
}

// The chunk of scan lane g: its sequence x (binary search over cbase) and
// chunk c within it.  Returns false past the last chunk.
__device__ __forceinline__ bool nuc_chunk(const NucArgs &a, int64_t g, int &x, int &c) {
    if (g >= a.nchunk) return false;
    int lo = 0, hi = a.nseq - 1;   // last x with cbase[x] <= g
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.cbase[mid] <= g) lo = mid;
        else hi = mid - 1;
    }
    x = lo;
    c = (int)(g - a.cbase[x]);
    return true;
}

// fn(q, p) for every match with start p in chunk c of sequence x, in order
// of p.  Bytes come four at a time from aligned words (a word holding a byte
// of the sequence never leaves its page).
template <class Fn>
__device__ __forceinline__ void nuc_scan_chunk(const NucArgs &a, const unsigned long long *tk, const int32_t *ts,
                                               int x, int c, Fn fn) {
    const int64_t so = a.off[x];
    const int n = (int)(a.off[x + 1] - so);
    const int k = a.k;
    const int p0 = c * kNucChunk, j1 = min(n, p0 + kNucChunk + k - 1);
    const uintptr_t a0 = (uintptr_t)(a.res + so + p0);
    const uint32_t *w = reinterpret_cast<const uint32_t *>(a0 & ~(uintptr_t)3);
    const int sh0 = (int)(a0 & 3);
    unsigned long long key = 0;
    int valid = 0;
    uint32_t word = p0 < j1 ? w[0] : 0u;
    for (int j = p0; j < j1; ++j) {
        const int at = sh0 + (j - p0);
        if (j > p0 && (at & 3) == 0) word = w[at >> 2];
        const uint32_t b = (word >> (8 * (at & 3))) & 0xffu;
        if (b > 3) {
            valid = 0;
            continue;
        }
        key = (key >> 2) | ((unsigned long long)b << (2 * (k - 1)));   // base j - k + 1 + t at bits 2t
        if (++valid >= k) {
            const int q = nuc_lookup(tk, ts, a.lg_t, key);
            if (q >= 0) fn(q, j - k + 1);
        }
    }
}

constexpr int kNucWaveMaxK = 29;   // the wavefront scan's window: k + 3 bases in 64 bits

// The match starts p = p0 + 4 lane + r (r < 4) of chunk c of a sequence (its
// residues at so, n of them), the
// lanes of a wavefront sharing the chunk: returns q_r (the segment, or -1) in
// q[r].  The chunk's bytes come in coalesced aligned words (one per lane, nine
// more for the last k - 1 bases), are realigned to the chunk's start, turned
// into 2-bit codes plus an invalid bit per base, and each lane gathers the
// codes of its 32 bases (4 lane .. 4 lane + 31) from the next seven lanes (20 bases
// and four lanes with 32-bit keys).
template <typename K>
__device__ __forceinline__ void nuc_scan_wave(const NucArgs &a, const K *tk, const int32_t *ts,
                                              int64_t so, int n, int c, int lane, int q[4]) {
    const int k = a.k;
    const int p0 = c * kNucChunk;
    const uint8_t *base = a.res + so;
    const uintptr_t ad = (uintptr_t)(base + p0);
    const uintptr_t A = ad & ~(uintptr_t)3;
    const uint32_t sh = (uint32_t)(ad & 3);
    const uintptr_t lim = (uintptr_t)(base + n);   // a word starting before it holds a byte of the sequence
    const uint32_t d0 = A + 4 * (uintptr_t)lane < lim ? *reinterpret_cast<const uint32_t *>(A + 4 * lane) : 0u;
    const uint32_t d1 =
        (lane < 9 && A + 256 + 4 * (uintptr_t)lane < lim) ? *reinterpret_cast<const uint32_t *>(A + 256 + 4 * lane) : 0u;
    // bytes p0 + 4 lane .. + 3 (e0) and p0 + 256 + 4 lane .. + 3 (e1, lanes < 8)
    const uint32_t n0 = __shfl(d0, (lane + 1) & 63, 64), n1 = __shfl(d1, 0, 64), n1b = __shfl(d1, (lane + 1) & 63, 64);
    const uint32_t e0 = (uint32_t)((((uint64_t)(lane < 63 ? n0 : n1) << 32) | d0) >> (8 * sh));
    const uint32_t e1 = (uint32_t)((((uint64_t)n1b << 32) | d1) >> (8 * sh));
    auto codes = [](uint32_t e) __attribute__((always_inline)) -> uint32_t {   // 2-bit codes | invalid bits << 8
        uint32_t v = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t b = (e >> (8 * j)) & 255u;
            v |= (b & 3u) << (2 * j);
            v |= (uint32_t)(b > 3u) << (8 + j);
        }
        return v;
    };
    const uint32_t ca = codes(e0), cb = codes(e1);
    uint64_t W = 0;   // base 4 lane + t at bits 2t
    uint32_t V = 0;   // its invalid bit at bit t
#pragma unroll
    for (int d = 0; d < (sizeof(K) == 4 ? 5 : 8); ++d) {   // k + 3 bases
        const int src = lane + d;
        const uint32_t va = __shfl(ca, src & 63, 64), vb = __shfl(cb, src & 63, 64);
        const uint32_t v = src < 64 ? va : vb;
        W |= (uint64_t)(v & 255u) << (8 * d);
        V |= (v >> 8) << (4 * d);
    }
    const uint64_t kmask = (1ull << (2 * k)) - 1ull;
    const uint32_t vmask = (1u << k) - 1u;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int p = p0 + 4 * lane + r;
        const bool ok = p + k <= n && ((V >> r) & vmask) == 0u;
        q[r] = ok ? nuc_lookup(tk, ts, a.lg_t, (K)((W >> (2 * r)) & kmask)) : -1;
    }
}

static_assert(kNucChunk == 4 * 64, "the wavefront scan takes four match starts per lane");

// Scan, wavefront form (k <= kNucWaveMaxK): the matches of every chunk, in
// order of p, and their number.  Each sequence's chunks are shared by a.wparts
// wavefronts.  One pass that stores (a chunk has at most kNucChunk matches, so each
// has its own place) instead of one that counts and one that stores: 105 us for both,
// and a search for each wavefront's sequence, at 672 x 16,569.
// Bound by VALU issue (about 370 instructions a chunk, half of them probes), not by
// its loads: with the next chunk's words loaded ahead it took as long.
template <typename K>
__global__ void __launch_bounds__(1024) nuc_scan_wave_kernel(NucArgs a) {
    NUC_TABLE_SETUP(K)   // shared by the workgroup's 16 wavefronts
    const int lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1ull;
    const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6), items = (int64_t)a.nseq * a.wparts;
    for (int64_t w = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); w < items; w += nw) {
        const int x = (int)(w / a.wparts), part = (int)(w - (int64_t)x * a.wparts);
        const int64_t cb = a.cbase[x], so = a.off[x];
        const int nc = (int)(a.cbase[x + 1] - cb), n = (int)(a.off[x + 1] - so);
        const int per = (nc + a.wparts - 1) / a.wparts, c1 = min(nc, (part + 1) * per);
        for (int c = part * per; c < c1; ++c) {
            int q[4];
            nuc_scan_wave(a, tk, ts, so, n, c, lane, q);
            int before = 0, total = 0;   // matches of the lanes below, of all
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint64_t b = __ballot(q[r] >= 0);
                before += __popcll(b & below);
                total += __popcll(b);
            }
            uint32_t *out = a.cmatch + so + (int64_t)c * kNucChunk + before;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (q[r] >= 0) *out++ = (uint32_t)q[r] << 8 | (uint32_t)(4 * lane + r);
            if (lane == 0) a.ccount[cb + c] = total;
        }
    }
}

// Scan, one lane per chunk (any k).
__global__ void __launch_bounds__(256) nuc_scan_kernel(NucArgs a) {
    NUC_TABLE_SETUP(unsigned long long)
    int x, c;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (!nuc_chunk(a, g, x, c)) return;
    uint32_t *out = a.cmatch + a.off[x] + (int64_t)c * kNucChunk;
    int cnt = 0;
    nuc_scan_chunk(a, tk, ts, x, c, [&](int q, int p) { out[cnt++] = (uint32_t)q << 8 | (uint32_t)(p - c * kNucChunk); });
    a.ccount[g] = cnt;
}

// Third pass: the anchor chain over a sequence's matches (in order of p).  A
// match is inserted into the chain table once p_i >= p_j + k for the match i
// being queried; tails[L] is the inserted match of chain length L with the
// smallest (q, p) (q increases with L).  A query takes the longest L whose
// tail has q < q_i: best = L + 1, predecessor = tails[L].  Sequential in the
// matches; returns L with the chain in tails[0 .. L-1].
//
// One lane walks it, so each dependent read is a trip to LDS (about 130 cycles).  Most
// matches follow the one before (q larger, p at least k further) and extend the
// longest chain, each inserted when the next one is queried: eight such
// matches are taken at once, on independent reads, and so are eight
// links of the chain that lead to the match before (one stray match makes a
// segment of up to all the matches it spans: 10 us at 1,000).
template <typename TM, typename TI>
__device__ __forceinline__ int nuc_chain_seq(const TM *mq, const TM *mp, TI *mbest, TI *mpred, TI *tails, int cnt,
                                             int k) {
    int L = 0, ins_next = 0;
    int lastq = -1, lastj = 0;   // q and index of tails[L]
    // the previous match's fields stay in registers: it is usually the next
    // one inserted (matches lie about k apart in p)
    int qprev = 0, pprev = 0, bprev = 0;
    int qn = cnt > 0 ? (int)mq[0] : 0, pn = cnt > 0 ? (int)mp[0] : 0;
    int again = 0;   // the next match from which eight at once are tried
    for (int i = 0; i < cnt; ++i) {
        if (i > again && i + 8 <= cnt && ins_next == i - 1 && bprev == L + 1) {
            int q8[8], p8[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                q8[u] = (int)mq[i + u];
                p8[u] = (int)mp[i + u];
            }
            bool follow = q8[0] > qprev && p8[0] >= pprev + k;
#pragma unroll
            for (int u = 1; u < 8; ++u) follow = follow && q8[u] > q8[u - 1] && p8[u] >= p8[u - 1] + k;
            if (follow) {   // i - 1 .. i + 6 inserted, i + 7 queried
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    tails[L + 1 + u] = (TI)(i - 1 + u);
                    mpred[i + u] = (TI)(i - 1 + u);
                }
                L += 8;
                lastq = q8[6];
                lastj = i + 6;
                ins_next = i + 7;
                mbest[i + 7] = (TI)(L + 1);
                qprev = q8[7];
                pprev = p8[7];
                bprev = L + 1;
                i += 7;
                if (i + 1 < cnt) {
                    qn = (int)mq[i + 1];
                    pn = (int)mp[i + 1];
                }
                continue;
            }
            again = i + 8;
        }
        const int q = qn, p = pn;
        if (i + 1 < cnt) {   // the next match's fields, loaded a match ahead
            qn = (int)mq[i + 1];
            pn = (int)mp[i + 1];
        }
        while (ins_next < i) {
            const bool reg = ins_next == i - 1;
            const int pj = reg ? pprev : (int)mp[ins_next];
            if (pj + k > p) break;
            const int j = ins_next++;
            const int bj = reg ? bprev : (int)mbest[j];
            const int qj = reg ? qprev : (int)mq[j];
            if (bj > L) {
                tails[bj] = (TI)j;
                L = bj;
                lastq = qj;
                lastj = j;
            } else if (qj < (int)mq[tails[bj]]) {
                tails[bj] = (TI)j;
                if (bj == L) {
                    lastq = qj;
                    lastj = j;
                }
            }
        }
        int lq = 0, pred = 0;   // pred unused for lq = 0
        if (L > 0 && lastq < q) {
            lq = L;
            pred = lastj;
        } else {
            int lo = 1, hi = L;   // largest l in [1, L] with q(tails[l]) < q
            while (lo <= hi) {
                const int mid = (lo + hi) >> 1;
                if ((int)mq[tails[mid]] < q) { lq = mid; lo = mid + 1; }
                else hi = mid - 1;
            }
            if (lq > 0) pred = (int)tails[lq];
        }
        mbest[i] = (TI)(lq + 1);
        mpred[i] = (TI)pred;
        qprev = q;
        pprev = p;
        bprev = lq + 1;
    }
    while (ins_next < cnt) {
        const int j = ins_next++;
        const int bj = (int)mbest[j];
        const int qj = (int)mq[j];
        if (bj > L) {
            tails[bj] = (TI)j;
            L = bj;
        } else if (qj < (int)mq[tails[bj]]) {
            tails[bj] = (TI)j;
        }
    }
    // the chain, in order, into tails[0 .. L-1] (tails[L] is its last match)
    int e = L > 0 ? (int)tails[L] : 0;
    again = L;
    for (int t = L - 1; t >= 0; --t) {
        if (t < again && t >= 8 && e >= 8) {
            bool run = true;
            int pr[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) pr[u] = (int)mpred[e - u];
#pragma unroll
            for (int u = 0; u < 8; ++u) run = run && pr[u] == e - u - 1;
            if (run) {
#pragma unroll
                for (int u = 0; u < 8; ++u) tails[t - u] = (TI)(e - u);
                t -= 7;
                e -= 8;
                continue;
            }
            again = t - 8;
        }
        tails[t] = (TI)e;
        e = (int)mpred[e];
    }
    return L;
}

constexpr int kChainLdsMax = 4096;   // matches of a sequence chained in LDS at most

// LDS of the chain kernel (16-bit units): q, p, best, pred [cap] each, tails
// [2 cap + 2], cut flags (bytes) [cap], then the aligned words (4-byte aligned)
__host__ __device__ inline size_t nuc_chain_lal_off(int cap) { return ((6 * (size_t)cap + 2 + ((size_t)cap + 1) / 2) + 1) & ~(size_t)1; }
inline size_t nuc_chain_lds_bytes(int cap, int aw) { return 2 * nuc_chain_lal_off(cap) + 4 * (size_t)aw; }

// The matrix in LDS, 32 x 32 with zeros past the alphabet.
#define NUC_SMAT_SETUP                                                              \
    __shared__ int8_t smat[32 * 32];                                                \
    for (int x_ = threadIdx.x; x_ < 1024; x_ += blockDim.x) {                       \
        const int r_ = x_ >> 5, q_ = x_ & 31;                                       \
        smat[x_] = (r_ < a.alpha && q_ < a.alpha) ? a.mat[r_ * a.alpha + q_] : (int8_t)0; \
    }                                                                               \
    __syncthreads();

// Inclusive prefix sum over a 256-lane workgroup, and the total (s4: four ints
// of LDS, free again after the caller's next barrier).
__device__ __forceinline__ int nuc_block_sum(int v, int *s4, int tid, int &total) {
    const int lane = tid & 63, w = tid >> 6;
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(v, d, 64);
        if (lane >= d) v += t;
    }
    if (lane == 63) s4[w] = v;
    __syncthreads();
    for (int u = 0; u < 4; ++u)
        if (u < w) v += s4[u];
    total = s4[0] + s4[1] + s4[2] + s4[3];
    return v;
}

// One 256-lane workgroup per sequence.  A sequence with at most a.chain_cap
// matches has them staged in LDS (q, p < 65536 as 16-bit fields) and chained
// there, segment by segment (below); a larger one is chained by lane 0 in
// global arrays.
//
// Then the lanes share the stretches (before the first anchor, between anchors,
// after the last), and settle here what needs no dynamic program:
//  - one side empty: a single gap;
//  - both sides of one length, and the plain diagonal scores at least as much as any
//    path with gaps could.  Such a path has a gap on either side, each of
//    which costs at least go + ge, and leaves a center base unaligned, so with r+ the
//    larger of 0 and a base's best score it stays at or under
//    sum r+ - min r+ - 2 (go + ge).  The diagonal is then an optimum, and
//    the one that the traceback takes (it prefers the diagonal in every cell).
// Substitutions cause most stretches: of about 34,000 in 672 genomes of 16,569
// bases, most end here (one lane each before, 159 us, and a wavefront each for the
// wide ones, 112 us).  The rest go to the lists, with their scratch.
__global__ void __launch_bounds__(256) nuc_chain_kernel(NucArgs a) {
    extern __shared__ uint16_t chain_lds[];
    NUC_SMAT_SETUP
    __shared__ int s_rmax[32], s_coff[257], s4[4], s4b[4], sh_L, sh_todo, sh_keep, sh_part;
    __shared__ long long sh_big;
    const int cap = a.chain_cap;
    uint16_t *lq = chain_lds, *lp = lq + cap, *lbest = lp + cap, *lpred = lbest + cap, *ltails = lpred + cap;
    uint8_t *lcut = reinterpret_cast<uint8_t *>(ltails + 2 * cap + 2);
    uint32_t *lal = reinterpret_cast<uint32_t *>(chain_lds + nuc_chain_lal_off(cap));   // [aw]: the aligned bits
    const int x = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t so = a.off[x];
    const int n = (int)(a.off[x + 1] - so);
    const int k = a.k, m = a.m, goe = a.go + a.ge;
    const bool own = a.own_row && x == a.gskip;
    const int64_t cb = a.cbase[x];
    const int nc = (int)(a.cbase[x + 1] - cb);   // at most 256 (n < 65536)
    if (tid < 32) {   // each base's best score, at least 0
        int r = 0;
        for (int q = 0; q < a.alpha; ++q) r = max(r, (int)smat[tid * 32 + q]);
        s_rmax[tid] = r;
    }
    if (tid == 0) {
        sh_todo = 0;
        sh_keep = 0;
        sh_part = 0;
    }
    for (int w = tid; w < a.aw; w += 256) lal[w] = 0u;
    const int cv = tid < nc ? a.ccount[cb + tid] : 0;
    int cnt;
    s_coff[tid + 1] = nuc_block_sum(cv, s4, tid, cnt);
    if (tid == 0) s_coff[0] = 0;
    const bool inl = cnt <= cap;
    if (!inl && tid == 0) sh_big = (long long)atomicAdd(a.count + kNucBig, (unsigned long long)cnt + 2);
    __syncthreads();
    const bool room = inl || sh_big + cnt + 2 <= a.bigcap;   // else the call runs this kernel again
    int32_t *gq = a.big + (inl ? 0 : sh_big), *gp = gq + a.bigcap, *gbest = gp + a.bigcap, *gpred = gbest + a.bigcap,
            *gtails = gpred + a.bigcap;
    if (room) {
        for (int c = tid >> 4; c < nc; c += 16) {
            const int at = s_coff[c], e = s_coff[c + 1] - at;
            const uint32_t *src = a.cmatch + so + (int64_t)c * kNucChunk;
            for (int i = tid & 15; i < e; i += 16) {
                const uint32_t v = src[i];
                const int q = (int)(v >> 8), p = c * kNucChunk + (int)(v & 255u);
                if (inl) {
                    lq[at + i] = (uint16_t)q;
                    lp[at + i] = (uint16_t)p;
                } else {
                    gq[at + i] = q;
                    gp[at + i] = p;
                }
            }
        }
    }
    __threadfence_block();
    __syncthreads();
    auto qof = [&](int j) __attribute__((always_inline)) -> int { return inl ? (int)lq[j] : gq[j]; };
    auto pof = [&](int j) __attribute__((always_inline)) -> int { return inl ? (int)lp[j] : gp[j]; };
    // When every match follows the one before it (q larger, p at least k
    // further), all of them form the one chain of length cnt, which is then
    // the longest: checked by all lanes, no sequential pass.
    bool ok = true;
    if (room)
        for (int i = tid; i + 1 < cnt; i += 256) ok = ok && qof(i + 1) > qof(i) && pof(i + 1) >= pof(i) + k;
    const bool ident = __syncthreads_and(ok) != 0;
    if (room && !ident && !inl) {
        if (tid == 0) sh_L = nuc_chain_seq(gq, gp, gbest, gpred, gtails, cnt, k);
        __threadfence_block();
    } else if (room && !ident) {
        // Cuts: b splits the matches when every match before it precedes every
        // match from it on (max q before b < min q from b, p[b-1] + k <= p[b]).
        // Then every match before b is inserted before b is queried, each query
        // from b on finds the prefix's whole chain below its q, and later
        // inserts touch only longer lengths: the chain is the prefix's chain
        // followed by the rest's.  So each segment between cuts is chained on
        // its own (lanes take the segments starting in their block), and the
        // segments' chains are joined in order.
        const int per = (cnt + 255) / 256, lo = min(cnt, tid * per), hi = min(cnt, lo + per);
        int bmax = -1, bmin = 0x7fffffff;
        for (int i = lo; i < hi; ++i) {
            bmax = max(bmax, (int)lq[i]);
            bmin = min(bmin, (int)lq[i]);
        }
        int pm = bmax, sm = bmin;   // inclusive prefix max, suffix min over the lanes
        for (int d = 1; d < 64; d <<= 1) {
            const int t1 = __shfl_up(pm, d, 64), t2 = __shfl_down(sm, d, 64);
            if (lane >= d) pm = max(pm, t1);
            if (lane + d < 64) sm = min(sm, t2);
        }
        if (lane == 63) s4[wv] = pm;
        if (lane == 0) s4b[wv] = sm;
        __syncthreads();
        int runmax = __shfl_up(pm, 1, 64), runmin = __shfl_down(sm, 1, 64);
        if (lane == 0) runmax = -1;
        if (lane == 63) runmin = 0x7fffffff;
        for (int u = 0; u < 4; ++u) {
            if (u < wv) runmax = max(runmax, s4[u]);
            if (u > wv) runmin = min(runmin, s4b[u]);
        }
        for (int i = hi - 1; i >= lo; --i) {   // min q from i on (lbest as scratch)
            runmin = min(runmin, (int)lq[i]);
            lbest[i] = (uint16_t)runmin;
        }
        for (int i = lo; i < hi; ++i) {
            lcut[i] = (i == 0 || (runmax < (int)lbest[i] && (int)lp[i - 1] + k <= (int)lp[i])) ? 1 : 0;
            runmax = max(runmax, (int)lq[i]);
        }
        __syncthreads();
        for (int b = lo; b < hi; ++b) {
            if (!lcut[b]) continue;
            int e = b + 1;
            while (e < cnt && !lcut[e]) ++e;
            const int Ls = nuc_chain_seq(lq + b, lp + b, lbest + b, lpred + b, ltails + 2 * b, e - b, k);
            lbest[b] = (uint16_t)Ls;   // the segment's chain length (its own best no longer needed)
        }
        __syncthreads();
        int sl = 0;
        for (int b = lo; b < hi; ++b)
            if (lcut[b]) sl += lbest[b];
        int total;
        int o = nuc_block_sum(sl, s4, tid, total) - sl;
        for (int b = lo; b < hi; ++b) {   // the chain, in order, into lpred (preds no longer needed)
            if (!lcut[b]) continue;
            const int Ls = lbest[b];
            for (int t = 0; t < Ls; ++t) lpred[o + t] = (uint16_t)(b + ltails[2 * b + t]);
            o += Ls;
        }
        if (tid == 0) sh_L = total;
    }
    __syncthreads();
    const int L = !room ? -1 : (ident ? cnt : sh_L);
    auto anchor = [&](int t) __attribute__((always_inline)) -> int {   // match index of anchor t < L
        return ident ? t : (inl ? (int)lpred[t] : gtails[t]);
    };
    const uint64_t below = (1ull << lane) - 1ull;   // lanes under this one
    // slot t of the chain (t <= L): the stretch from just past anchor t - 1 to
    // anchor t (or the ends)
    auto stretch = [&](int t, int &ci, int &sj, int &dc, int &ds, int &jt) __attribute__((always_inline)) {
        ci = 0;
        sj = 0;
        if (t > 0) {
            const int jp = anchor(t - 1);
            ci = qof(jp) * k + k;
            sj = pof(jp) + k;
        }
        jt = t < L ? anchor(t) : 0;
        dc = (t < L ? qof(jt) * k : m) - ci;
        ds = (t < L ? pof(jt) : n) - sj;
    };
    auto set_bits = [&](int p0, int len) __attribute__((always_inline)) {   // center positions aligned
        for (int w = p0 >> 5; w <= (p0 + len - 1) >> 5; ++w) {
            const int b0 = max(p0, w << 5) - (w << 5), b1 = min(p0 + len, (w + 1) << 5) - (w << 5);
            atomicOr(lal + w, (b1 - b0 == 32) ? ~0u : (((1u << (b1 - b0)) - 1u) << b0));
        }
    };
    // the diagonal's score, if it is settled (kNucNeg otherwise); four lanes
    // share a stretch, each four of every 16 bases, from aligned words (a word
    // holding a byte of the stretch never leaves its page)
    auto diagonal = [&](bool test, int ci, int sj, int len) __attribute__((always_inline)) -> int {
        const uintptr_t ac = (uintptr_t)(a.center + ci), as = (uintptr_t)(a.res + so + sj);
        const uint32_t *wc = reinterpret_cast<const uint32_t *>(ac & ~(uintptr_t)3);
        const uint32_t *ws = reinterpret_cast<const uint32_t *>(as & ~(uintptr_t)3);
        const int hc = (int)(ac & 3), hs = (int)(as & 3);
        const int nwc = (hc + len + 3) >> 2, nws = (hs + len + 3) >> 2;   // words that hold the stretch
        int diag = 0, best = 0, least = 0x7fffffff;
        for (int i0 = 4 * (lane & 3); test && i0 < len; i0 += 16) {
            const int w = i0 >> 2;
            const uint32_t c0 = w < nwc ? wc[w] : 0u, c1 = w + 1 < nwc ? wc[w + 1] : 0u;
            const uint32_t s0 = w < nws ? ws[w] : 0u, s1 = w + 1 < nws ? ws[w + 1] : 0u;
            const uint32_t c4 = (uint32_t)(((uint64_t)c1 << 32 | c0) >> (8 * hc));
            const uint32_t s4w = (uint32_t)(((uint64_t)s1 << 32 | s0) >> (8 * hs));
            int sc[4], rm[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int cc = (int)(c4 >> (8 * b)) & 31;
                sc[b] = smat[cc * 32 + ((int)(s4w >> (8 * b)) & 31)];
                rm[b] = s_rmax[cc];
            }
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (i0 + b < len) {
                    diag += sc[b];
                    best += rm[b];
                    least = min(least, rm[b]);
                }
        }
#pragma unroll
        for (int o = 1; o <= 2; o <<= 1) {
            diag += __shfl_xor(diag, o, 64);
            best += __shfl_xor(best, o, 64);
            least = min(least, __shfl_xor(least, o, 64));
        }
        return test && diag >= best - least - 2 * goe ? diag : kNucNeg;
    };
    int part = 0;   // this lane's share of the score
    // stretch t (neither side empty) of each lane that asks, into the lists, with
    // its scratch; the whole wavefront comes here together
    auto list = [&](bool act, int t) __attribute__((always_inline)) {
        int ci = 0, sj = 0, dc = 0, ds = 0, jt = 0;
        if (act) stretch(t, ci, sj, dc, ds, jt);
        if (__ballot(act) == 0) return;
        const bool wide = act && (ds > kNucSmallW || dc > kNucTallH);
        const bool tiny = act && !wide && dc <= kNucTinyW && ds <= kNucTinyW;
        const bool sm = act && !wide && !tiny;
        const uint64_t bt = __ballot(tiny), bs = __ballot(sm), bw = __ballot(wide);
        const int64_t rneed = wide ? dc + 1 : 0;   // the wavefront's boundary column
        const int64_t cneed = act ? (int64_t)dc * ((ds + 7) >> 3) : 0;
        int64_t ri = rneed, ki = cneed;   // inclusive sums over the lanes
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t t1 = __shfl_up(ri, d, 64), t2 = __shfl_up(ki, d, 64);
            if (lane >= d) {
                ri += t1;
                ki += t2;
            }
        }
        // one atomic per counter, on lanes of their own
        unsigned long long got = 0;
        const unsigned long long radd = (unsigned long long)__shfl(ri, 63, 64), kadd = (unsigned long long)__shfl(ki, 63, 64);
        if (lane < 4) {
            const unsigned long long add =
                lane == 0   ? radd
                : lane == 1 ? kadd
                : lane == 2 ? (unsigned long long)__popcll(bt) | (unsigned long long)__popcll(bs) << 32
                            : (unsigned long long)__popcll(bw);
            if (add) got = atomicAdd(a.count + 32 * lane, add);   // kNucRows, kNucCodes, kNucNarrow, kNucWide
        }
        const int64_t r0 = (int64_t)__shfl((long long)got, 0, 64), k0 = (int64_t)__shfl((long long)got, 1, 64);
        const unsigned long long nn = (unsigned long long)__shfl((long long)got, 2, 64);
        const int64_t w0 = (int64_t)__shfl((long long)got, 3, 64);
        if (!act) return;
        const int64_t at = wide ? w0 + __popcll(bw & below)
                           : tiny ? (int64_t)(nn & 0xffffffffull) + __popcll(bt & below)
                                  : a.listcap - 1 - ((int64_t)(nn >> 32) + __popcll(bs & below));
        if (at < 0 || at >= a.listcap) return;   // (the call runs this kernel again)
        const longlong2 off = make_longlong2(r0 + ri - rneed, k0 + ki - cneed);
        (wide ? a.wd : a.nd)[at] = make_int4(ci, dc, sj, ds);
        (wide ? a.wx : a.nx)[at] = x;
        (wide ? a.wo : a.no)[at] = off;
    };
    uint16_t *todo = ltails, *keep = ltails + cap + 1;   // (free by now; each with room for cap + 1 slots)
    for (int t0 = 0; t0 <= L; t0 += 256) {   // uniform trip count (ballots)
        const int t = t0 + tid;
        int ci = 0, sj = 0, dc = 0, ds = 0, jt = 0;
        if (t <= L) stretch(t, ci, sj, dc, ds, jt);
        if (t < L) {   // the anchor
            set_bits(ci + dc, k);
            part += a.segscore[qof(jt)];
        }
        const bool gap = t <= L && (dc == 0) != (ds == 0);
        if (gap) part -= a.go + a.ge * (dc + ds);
        if (gap && ds > 0 && !own) {   // residues inserted after center position ci
            a.ins[(int64_t)x * (m + 1) + ci] = (uint16_t)ds;
            if (a.G && x != a.gskip) atomicMax(a.G + ci, ds);
        }
        const bool work = t <= L && dc > 0 && ds > 0;
        if (!inl) continue;
        const uint64_t b = __ballot(work);
        int at = 0;
        if (lane == 0 && b) at = atomicAdd(&sh_todo, __popcll(b));
        at = __shfl(at, 0, 64);
        if (work) todo[at + __popcll(b & below)] = (uint16_t)t;
    }
    __syncthreads();
    const int ntodo = inl ? sh_todo : L + 1;   // (a larger sequence's slots are all looked at again)
    for (int i0 = 16 * wv; i0 < ntodo; i0 += 64) {   // four lanes a stretch
        const int i = i0 + (lane >> 2);
        bool act = i < ntodo;
        const int t = act ? (inl ? (int)todo[i] : i) : 0;
        int ci = 0, sj = 0, dc = 0, ds = 0, jt = 0;
        if (act) stretch(t, ci, sj, dc, ds, jt);
        const int v = diagonal(act && dc == ds && dc <= kNucDiagMax, ci, sj, dc);
        act = act && dc > 0 && ds > 0 && (lane & 3) == 0;   // one lane goes on
        if (act && v != kNucNeg) {
            part += v;
            set_bits(ci, dc);
            act = false;
        }
        if (!inl) list(act, t);
        else if (act) keep[atomicAdd(&sh_keep, 1)] = (uint16_t)t;
    }
    // a sequence's stretches listed together: an atomic per counter and
    // sequence (one per 16 stretches took 24 us of waiting, all on one line)
    __syncthreads();
    if (inl && wv == 0)
        for (int i0 = 0; i0 < sh_keep; i0 += 64) list(i0 + lane < sh_keep, i0 + lane < sh_keep ? (int)keep[i0 + lane] : 0);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) part += __shfl_xor(part, o, 64);
    if (lane == 0) atomicAdd(&sh_part, part);
    __syncthreads();
    uint32_t *al = a.aligned + (int64_t)x * a.aw;
    for (int w = tid; w < a.aw; w += 256)   // stretches OR in later
        al[w] = own ? (32 * w + 32 <= m ? ~0u : (1u << (m & 31)) - 1u) : lal[w];
    if (tid != 0) return;
    a.score[x] = sh_part;
    if (!a.mail) return;
    // The last workgroup tells the host.  Only the counts have to be there, and
    // every workgroup has its atomics' results before its barrier above; a
    // device-wide fence, which writes the caches back, took 28 us here.
    if (atomicAdd(a.count + kNucDone, 1ull) + 1 != gridDim.x) return;
    for (int c = 0; c < 5; ++c)
        __hip_atomic_store(a.mail + 3 + c,
                           (int64_t)__hip_atomic_load(a.count + 32 * c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(a.mail + 2, (int64_t)*a.flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(a.mail + 1, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Last pass: each listed stretch aligned end to end (Gotoh's global form,
// H(0,0) = 0, H(i,0) = -(go + ge*i), H(0,j) = -(go + ge*j), E(i,0) = F(0,j) =
// -inf), codes per cell (bit 0 diagonal not taken, 1 E not taken, 2 E
// extended, 3 F extended; eight cells per word, cw = ceil(ds / 8) words a
// row), then the traceback with the local alignment's priorities into the
// center-star vector.  Stretches of a sequence touch disjoint insertion slots;
// aligned words and the score are shared (atomics).

// The traceback from (dc, ds) to (0, 0) over a stretch's codes (word w at
// code(w)): diagonal steps mark center positions aligned, E steps count residues
// into the insertion slot after their center position (a slot's count is written
// once, with the merge's running max).
template <class Code>
__device__ __forceinline__ void nuc_traceback(const NucArgs &a, int x, int ci, int dc, int ds, Code code) {
    const int cw = (ds + 7) >> 3;
    uint16_t *ins = a.ins + (int64_t)x * (a.m + 1);
    uint32_t *al = a.aligned + (int64_t)x * a.aw;
    int32_t *gmax = (a.G && x != a.gskip) ? a.G : nullptr;
    const int go = a.go;
    int i = dc, j = ds, st = 0;   // 0 H, 1 E, 2 F
    int sl = -1, scount = 0;
    int curw = -1;
    uint32_t bits = 0;
    while (i > 0 || j > 0) {
        const uint32_t nib = (i > 0 && j > 0)
                                 ? (code((int64_t)(i - 1) * cw + ((j - 1) >> 3)) >> (4 * ((j - 1) & 7))) & 15u
                                 : 0u;
        if (st == 0) {
            if (i > 0 && j > 0) {
                if (!(nib & 1u)) {
                    const int p = ci + i - 1;
                    if ((p >> 5) != curw) {
                        if (curw >= 0) atomicOr(al + curw, bits);
                        curw = p >> 5;
                        bits = 0;
                    }
                    bits |= 1u << (p & 31);
                    --i;
                    --j;
                } else {
                    st = (nib & 2u) ? 2 : 1;
                }
            } else {
                st = i == 0 ? 1 : 2;
            }
        } else if (st == 1) {
            // s_j after center position ci + i: slot ci + i
            if (ci + i != sl) {
                if (sl >= 0) {
                    ins[sl] = (uint16_t)scount;
                    if (gmax) atomicMax(gmax + sl, scount);
                }
                sl = ci + i;
                scount = 0;
            }
            ++scount;
            const bool ext = (i > 0) ? (nib & 4u) != 0 : (j > 1 && go > 0);
            --j;
            if (!ext) st = 0;
        } else {
            const bool ext = (j > 0) ? (nib & 8u) != 0 : (i > 1 && go > 0);
            --i;
            if (!ext) st = 0;
        }
    }
    if (sl >= 0) {
        ins[sl] = (uint16_t)scount;
        if (gmax) atomicMax(gmax + sl, scount);
    }
    if (curw >= 0) atomicOr(al + curw, bits);
}

// A narrow stretch (at most kNucSmallW columns and kNucTallH rows) on one lane:
// the row of (H, F) sits in registers, the codes go to the stretch's code
// region, then the lane's traceback reads them back.
__device__ __forceinline__ void nuc_stretch_lane(const NucArgs &a, const int8_t *smat, bool act, int4 d, int x,
                                                 int64_t codeoff) {
    const int go = a.go, ge = a.ge, goe = go + ge;
    const int ci = d.x, dc = d.y, sj = d.z, ds = d.w;
    // the widest stretch of the wavefront bounds the unrolled columns
    int wmax = ds;
    for (int o = 32; o >= 1; o >>= 1) wmax = max(wmax, __shfl_xor(wmax, o, 64));
    wmax = __builtin_amdgcn_readfirstlane(wmax);
    const uint8_t *cc = a.center + ci, *ss = a.res + a.off[x] + sj;
    uint32_t *code0 = a.codes + codeoff;
    const int cw = (ds + 7) >> 3;
    uint32_t sw[kNucSmallW / 4];   // the stretch's residues, four per word
#pragma unroll
    for (int w = 0; w < kNucSmallW / 4; ++w) {
        uint32_t v = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int jj = 4 * w + b;
            if (jj < ds) v |= (uint32_t)(ss[jj] & 31) << (8 * b);
        }
        sw[w] = v;
    }
    int H[kNucSmallW + 1], F[kNucSmallW + 1];
#pragma unroll
    for (int j = 0; j <= kNucSmallW; ++j) {
        H[j] = j == 0 ? 0 : -(go + ge * j);
        F[j] = kNucNeg;
    }
    // the center's bases eight rows at a time, the next eight loaded a
    // group ahead
    auto load8 = [&](int i0) __attribute__((always_inline)) -> uint64_t {
        uint64_t v = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i0 + u < dc) v |= (uint64_t)(cc[i0 + u] & 31) << (8 * u);
        return v;
    };
    uint64_t cwin = load8(0), cnext = load8(8);
    for (int i = 1; i <= dc; ++i) {
        if (((i - 1) & 7) == 0 && i > 1) {
            cwin = cnext;
            cnext = load8(i + 7);
        }
        const int cr = (int)((cwin >> (8 * ((i - 1) & 7))) & 255u) * 32;
        int hdiag = H[0];
        int hleft = -(go + ge * i), eleft = kNucNeg;
        H[0] = hleft;
        uint32_t *crow = code0 + (int64_t)(i - 1) * cw;
        uint32_t word = 0;
#pragma unroll
        for (int j = 1; j <= kNucSmallW; ++j) {
            if (j > wmax) continue;   // uniform: past the wavefront's widest stretch
            const int e = max(eleft - ge, hleft - goe);
            const int f = max(F[j] - ge, H[j] - goe);
            const int dd = hdiag + smat[cr + ((sw[(j - 1) >> 2] >> (8 * ((j - 1) & 3))) & 255u)];
            const int h = max(dd, max(e, f));
            const uint32_t nib = (uint32_t)(h != dd) | ((uint32_t)(h != e) << 1) |
                                 ((uint32_t)(eleft - ge > hleft - goe) << 2) |
                                 ((uint32_t)(F[j] - ge > H[j] - goe) << 3);
            word |= nib << (4 * ((j - 1) & 7));
            if ((j & 7) == 0 || j == wmax) {
                if (((j - 1) >> 3) < cw) crow[(j - 1) >> 3] = word;
                word = 0;
            }
            hdiag = H[j];
            H[j] = h;
            F[j] = f;
            hleft = h;
            eleft = e;
        }
    }
    int hend = H[0];
#pragma unroll
    for (int j = 1; j <= kNucSmallW; ++j)
        if (j == ds) hend = H[j];
    if (act) {
        atomicAdd(a.score + x, hend);
        if (!(a.own_row && x == a.gskip)) nuc_traceback(a, x, ci, dc, ds, [&](int64_t w) { return code0[w]; });
    }
}

// The same traceback by a wavefront, all lanes at the same cell: the diagonal
// steps from a cell are read 64 at a time, and their bits set together.
template <class Code>
__device__ __forceinline__ void nuc_traceback_wave(const NucArgs &a, int lane, int x, int ci, int dc, int ds, Code code) {
    const int cw = (ds + 7) >> 3;
    uint16_t *ins = a.ins + (int64_t)x * (a.m + 1);
    uint32_t *al = a.aligned + (int64_t)x * a.aw;
    int32_t *gmax = (a.G && x != a.gskip) ? a.G : nullptr;
    const int go = a.go;
    auto nibble = [&](int i, int j) __attribute__((always_inline)) -> uint32_t {   // of cell (i, j), both > 0
        return (code((int64_t)(i - 1) * cw + ((j - 1) >> 3)) >> (4 * ((j - 1) & 7))) & 15u;
    };
    int i = dc, j = ds, st = 0;
    int sl = -1, scount = 0;
    auto flush = [&]() __attribute__((always_inline)) {
        if (sl >= 0 && lane == 0) {
            ins[sl] = (uint16_t)scount;
            if (gmax) atomicMax(gmax + sl, scount);
        }
    };
    while (i > 0 || j > 0) {
        if (st == 0) {
            if (i == 0 || j == 0) {
                st = i == 0 ? 1 : 2;
                continue;
            }
            const int len = min(64, min(i, j));
            const uint32_t nib = lane < len ? nibble(i - lane, j - lane) : 0u;
            const uint64_t stop = __ballot(lane < len && (nib & 1u));
            const int run = stop ? __builtin_ctzll(stop) : len;   // cells that take the diagonal
            if (run > 0) {   // at most three words of bits
                const int p0 = ci + i - run, w = (p0 >> 5) + lane;
                const int b0 = max(p0, w << 5) - (w << 5), b1 = min(p0 + run, (w + 1) << 5) - (w << 5);
                if (b1 > b0) atomicOr(al + w, (b1 - b0 == 32) ? ~0u : (((1u << (b1 - b0)) - 1u) << b0));
                i -= run;
                j -= run;
            }
            if (stop) st = ((uint32_t)__builtin_amdgcn_readlane((int)nib, run) & 2u) ? 2 : 1;
        } else if (st == 1) {
            const uint32_t nib = i > 0 ? nibble(i, j) : 0u;
            if (ci + i != sl) {
                flush();
                sl = ci + i;
                scount = 0;
            }
            ++scount;
            const bool ext = (i > 0) ? (nib & 4u) != 0 : (j > 1 && go > 0);
            --j;
            if (!ext) st = 0;
        } else {
            const uint32_t nib = j > 0 ? nibble(i, j) : 0u;
            const bool ext = (j > 0) ? (nib & 8u) != 0 : (i > 1 && go > 0);
            --i;
            if (!ext) st = 0;
        }
        i = __builtin_amdgcn_readfirstlane(i);
        j = __builtin_amdgcn_readfirstlane(j);
        st = __builtin_amdgcn_readfirstlane(st);
    }
    flush();
}

// v of the lane below (lane 0: first); inclusive prefix max over the 64 lanes
__device__ __forceinline__ int nuc_lane_below(int v, int first) {
    return __builtin_amdgcn_update_dpp(first, v, 0x138, 0xf, 0xf, false);   // wave_shr:1
}
__device__ __forceinline__ int wave_prefix_max(int v) {
    constexpr int kLeast = -0x7fffffff - 1;
    v = max(v, __builtin_amdgcn_update_dpp(kLeast, v, 0x111, 0xf, 0xf, false));   // row_shr:1, 2, 4, 8
    v = max(v, __builtin_amdgcn_update_dpp(kLeast, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(kLeast, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(kLeast, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(kLeast, v, 0x142, 0xa, 0xf, false));   // row_bcast:15
    v = max(v, __builtin_amdgcn_update_dpp(kLeast, v, 0x143, 0xc, 0xf, false));   // row_bcast:31
    return v;
}

constexpr int kNucCodeLds = 2048;   // code words of a stretch kept in LDS at most

// A stretch on a wavefront, in strips of 64 columns, lane L owning column 64 b +
// 1 + L of strip b and keeping (H, F) of the row above in registers.  E along a
// row is a max-plus scan: with Ht = max(D, F) and A(j) = Ht(i, j) + ge j,
//   E(i, j) + ge j = max(E(i, jb) + ge jb, H(i, jb) + ge jb - go,
//                        max over jb < j' < j of A(j') - go)
// for the strip's left boundary jb (since E - ge >= E - go - ge, extending from
// an E-derived H never beats the gap it continues).  The boundary column (H, E)
// per row passes from strip to strip through the stretch's row region
// (dc + 1 entries), 64 rows per coalesced load or store.  The row step is one
// dependent chain, so its exchanges between lanes are DPP moves rather than trips
// through LDS, and the codes stay in LDS where they fit: the traceback is a chain
// of reads.
__device__ __forceinline__ void nuc_stretch_wave(const NucArgs &a, const int8_t *smat, uint32_t *lcode, int lane, int4 d,
                                                 int x, int2 *bnd, uint32_t *gcode) {
    const int go = a.go, ge = a.ge, goe = go + ge;
    constexpr int kLow = -(1 << 30);
    const int ci = d.x, dc = d.y, sj = d.z, ds = d.w;
    const uint8_t *cc = a.center + ci, *ss = a.res + a.off[x] + sj;
    if (dc == ds && dc > kNucDiagMax) {   // the plain diagonal, as in the chain kernel
        int diag = 0, best = 0, least = 0x7fffffff;
        for (int i = lane; i < dc; i += 64) {
            const int c = cc[i] & 31, s = ss[i] & 31;
            int r = 0;
            for (int q = 0; q < a.alpha; ++q) r = max(r, (int)smat[c * 32 + q]);
            diag += smat[c * 32 + s];
            best += r;
            least = min(least, r);
        }
        for (int o = 32; o >= 1; o >>= 1) {
            diag += __shfl_xor(diag, o, 64);
            best += __shfl_xor(best, o, 64);
            least = min(least, __shfl_xor(least, o, 64));
        }
        if (diag >= best - least - 2 * goe) {
            uint32_t *al = a.aligned + (int64_t)x * a.aw;
            for (int w = (ci >> 5) + lane; w <= (ci + dc - 1) >> 5; w += 64) {
                const int b0 = max(ci, w << 5) - (w << 5), b1 = min(ci + dc, (w + 1) << 5) - (w << 5);
                atomicOr(al + w, (b1 - b0 == 32) ? ~0u : (((1u << (b1 - b0)) - 1u) << b0));   // (all set in an own row)
            }
            if (lane == 0) atomicAdd(a.score + x, diag);
            return;
        }
    }
    const int cw = (ds + 7) >> 3;
    const bool lc = dc * cw <= kNucCodeLds;   // (dc <= 65535, cw <= 8192)
    const int nstrip = (ds + 63) >> 6;
    for (int b = 0; b < nstrip; ++b) {
        const int jb = 64 * b;
        const int j = jb + 1 + lane;
        const bool inj = j <= ds;
        const int sres = inj ? ss[j - 1] & 31 : 0;
        int hp = -(go + ge * j), fp = kNucNeg;         // (H, F)(0, j)
        int bh_prev = b == 0 ? 0 : -(go + ge * jb);    // H(0, jb)
        const int w = 8 * b + (lane >> 3);
        const bool cst = (lane & 7) == 0 && w < cw;
        for (int i0 = 1; i0 <= dc; i0 += 64) {
            const int nr = min(64, dc - i0 + 1);
            const int2 ld = (b > 0 && lane < nr) ? bnd[i0 + lane] : make_int2(0, 0);
            const int crs = lane < nr ? cc[i0 - 1 + lane] & 31 : 0;
            int2 out = make_int2(0, 0);
            int snext = smat[__builtin_amdgcn_readlane(crs, 0) * 32 + sres];   // a row ahead
            for (int r = 0; r < nr; ++r) {
                const int i = i0 + r;
                const int sub = snext;
                snext = smat[__builtin_amdgcn_readlane(crs, (r + 1) & 63) * 32 + sres];
                const int bh = b == 0 ? -(go + ge * i) : __builtin_amdgcn_readlane(ld.x, r);   // H(i, jb)
                const int be = b == 0 ? kNucNeg : __builtin_amdgcn_readlane(ld.y, r);          // E(i, jb)
                const int hd = nuc_lane_below(hp, bh_prev);   // H(i-1, j-1)
                const int dd = hd + sub;
                const int f = max(fp - ge, hp - goe);
                const int ht = max(dd, f);
                const int inc = wave_prefix_max(ht + ge * j);
                const int ex = nuc_lane_below(inc, kLow);
                const int ehat = max(max(be + ge * jb, bh + ge * jb - go), ex - go);
                const int e = ehat - ge * j;
                const int h = max(ht, e);
                const int el = nuc_lane_below(e, be), hl = nuc_lane_below(h, bh);   // (E, H)(i, j-1)
                uint32_t nib = (uint32_t)(h != dd) | ((uint32_t)(h != e) << 1) |
                               ((uint32_t)(el - ge > hl - goe) << 2) | ((uint32_t)(fp - ge > hp - goe) << 3);
                if (!inj) nib = 0;
                // the eight lanes' codes in one word (lanes ^ 1, ^ 2, the other four)
                uint32_t v = nib << (4 * (lane & 7));
                v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, false);
                v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, false);
                v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false);   // row_half_mirror
                if (cst) {
                    if (lc) lcode[(i - 1) * cw + w] = v;
                    else gcode[(int64_t)(i - 1) * cw + w] = v;
                }
                const int oh = __builtin_amdgcn_readlane(h, 63), oe = __builtin_amdgcn_readlane(e, 63);   // (H, E)(i, jb + 64)
                if (lane == r) out = make_int2(oh, oe);
                if (i == dc && j == ds) atomicAdd(a.score + x, h);   // H(dc, ds)
                bh_prev = bh;
                hp = h;
                fp = f;
            }
            if (b + 1 < nstrip && lane < nr) bnd[i0 + lane] = out;
        }
        // the boundary column and the codes, before the next strip and the traceback read them
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
    }
    if (a.own_row && x == a.gskip) {
    } else if (lc) {
        nuc_traceback_wave(a, lane, x, ci, dc, ds, [&](int64_t w) { return lcode[w]; });
    } else {
        nuc_traceback_wave(a, lane, x, ci, dc, ds, [&](int64_t w) { return gcode[w]; });
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // and the reads before the next stretch's codes
    __builtin_amdgcn_wave_barrier();
}

// Narrow stretches take a lane each from this many on, a wavefront each below:
// a wavefront ends sooner, but takes more issue slots.  Whole calls, a lane each
// against a wavefront each: 3,600 stretches (672 genomes of 16,569) 356 against 264 us,
// 16,000 (3,000 genomes) 1,145 against 1,099, 32,000 (6,000) 2,093 against 2,188.
constexpr int64_t kNucLaneMin = 24576;

__global__ void __launch_bounds__(256) nuc_stretch_kernel(NucArgs a) {
    NUC_SMAT_SETUP
    __shared__ uint32_t s_code[4][kNucCodeLds];
    const unsigned long long nn = a.count[kNucNarrow], nwd = a.count[kNucWide];
    if (nuc_overflow(a, a.count[kNucRows], a.count[kNucCodes], nn, nwd, a.count[kNucBig])) return;
    const int64_t nt = (int64_t)(nn & 0xffffffffull), nnar = nt + (int64_t)(nn >> 32);   // the front's, and all
    auto place = [&](int64_t i) __attribute__((always_inline)) { return i < nt ? i : a.listcap - 1 - (i - nt); };
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const bool lanes = nnar >= a.lane_min;
    if (lanes)
        for (int64_t base = (int64_t)blockIdx.x * 256; base < nnar; base += (int64_t)gridDim.x * 256) {
            const int64_t i = base + threadIdx.x;
            const bool act = i < nnar;
            const int64_t at = act ? place(i) : 0;
            nuc_stretch_lane(a, smat, act, act ? a.nd[at] : make_int4(0, 0, 0, 0), act ? a.nx[at] : 0,
                             act ? (int64_t)a.no[at].y : 0);
        }
    const int64_t nsm = lanes ? 0 : nnar, items = (int64_t)nwd + nsm;
    for (int64_t it = (int64_t)blockIdx.x * 4 + wv; it < items; it += (int64_t)gridDim.x * 4) {
        const bool wide = it < (int64_t)nwd;   // the wide ones first
        const int64_t at = wide ? it : place(it - (int64_t)nwd);
        const int4 d = wide ? a.wd[at] : a.nd[at];
        const longlong2 o = wide ? a.wo[at] : a.no[at];
        nuc_stretch_wave(a, smat, s_code[wv], lane, d, wide ? a.wx[at] : a.nx[at], a.rows + o.x, a.codes + o.y);
    }
}

#undef NUC_SMAT_SETUP
#undef NUC_TABLE_SETUP

}  // namespace hk

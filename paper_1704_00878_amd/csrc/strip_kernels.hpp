// Strip kernel (one pair per lane) for gfx950: the score and traceback
// forward pass of many pairs against per-group centers.  Shares the
// recurrence, register form, traceback code and end-cell rule of the
// wavefront kernel (sw_kernels.hpp).
#pragma once
#include "sw_kernels.hpp"
#include "pk16.hpp"
#include "tiling.hpp"

namespace hk {

// ---------------------------------------------------------------------------
// Inter-task kernel: one pair per lane, 64 pairs per wavefront (one wave per
// workgroup, persistent over groups).  Lane-private state is a strip of T=16
// center rows; the wave sweeps j over the group's longest sequence, strip by
// strip.  The strip's profile (32 x 16 int32, stride 20) is rebuilt in LDS per
// strip from the group's center, so a group may use the batch center or any
// sequence of the set as its center (center selection, training targets).
// Strip boundaries (Hg, F* of the strip's last row for every j) go through a
// per-workgroup scratch row, read with agent-scope loads so that no stale L1
// line is seen.
//
// Codes: u64 (two u32 words: rows 0-7, 8-15; row t nibble at 4*(7 - t%8))
// per (strip s, column j, lane), tiled so that a lane's 4 consecutive columns
// share 32 bytes: with G = ceil(nmax/4),
//   codes[gbase + ((s*G + (j-1)/4)*64 + lane)*8 + ((j-1)%4)*2 + half].
// ---------------------------------------------------------------------------
constexpr int kT = 16;
constexpr int kPS = kT + 4;  // LDS row stride of the strip profile
constexpr int kB = 4;        // columns per prefetch block (the 4 columns of a code chunk)
constexpr int kFBits = 26, kFMask = (1 << kFBits) - 1;  // F* bits of a strip boundary cell (residue code above)

struct InterArgs {
    const int8_t *mat;
    int alpha;
    const uint8_t *center;    // batch center (mode 0)
    int m;
    const uint8_t *res;
    const int64_t *off;
    int mode;                 // 0 batch, 1 all pairs (a < b), 2 anchored groups
    const int32_t *order;     // mode 0: 64 * ngroups pair ids (-1 = empty lane); NULL: pair 64g + lane
    const int32_t *gnmax;     // mode 0: per group longest sequence (code layout); NULL: from the lanes
    const int32_t *gcen;      // mode 2: center seq id per group
    const int32_t *gb0;       // mode 2: first partner position in perm per group
    const int32_t *perm;      // modes 1/2: sequence ids (mode 1: sorted by length)
    int nseq;
    const int32_t *gslot;     // mode 2: sums slot of the group's center
    const int32_t *gorder;    // mode 1, 16-bit: the groups in running order (NULL: from the last one down)
    const int32_t *gcen2, *gslot2;   // the same of its second center (16-bit kernel; center -1: none)
    int64_t *sums;            // modes 1/2: integer score sums (atomic adds)
    int64_t ngroups;          // groups of this launch
    int64_t gfirst, gtotal;   // mode 1: this launch runs groups gfirst .. gfirst + ngroups - 1 of the
                              // gtotal = tri_groups(nseq, 64) or, 16-bit, pair_groups(nseq), largest first
    int ge, goe;
    unsigned long long *counter;   // next group (zeroed before the launch)
    int32_t *score;           // mode 0: per pair id; mode 2: per lane slot (optional)
    int32_t *endcell;         // mode 0: (i1, j1) per pair id (optional)
    int4 *cells4;             // mode 0 score-only: (0, 0, i1, j1) per pair id (optional)
    uint32_t *codes;
    const int64_t *gcode_base;// per group (u32 words)
    int2 *bound;              // per workgroup slot: bstride int2
    int64_t bstride;          // >= 64 * (max nmax rounded up to kB)
};

// a wave-uniform 64-bit value (read from LDS by every lane) in SGPRs
__device__ __forceinline__ int64_t uniform64(unsigned long long v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int2 load_agent(const int2 *p) {
    uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    return make_int2((int)(uint32_t)v, (int)(uint32_t)(v >> 32));
}

template <bool TB, bool ENDC>
__global__ void __launch_bounds__(64)
sw_inter_kernel(InterArgs a) {
    __shared__ int prof[(kAlphaMax + 1) * kPS];
    __shared__ uint32_t stage_all[64 * 8];
    __shared__ int8_t smat[kAlphaMax * kAlphaMax];
    const int lane = threadIdx.x;
    for (int x = lane; x < kAlphaMax * kAlphaMax; x += 64) {
        const int r = x >> 5, q = x & 31;
        smat[x] = (r < a.alpha && q < a.alpha) ? a.mat[r * a.alpha + q] : (int8_t)0;
    }
    int2 *bnd = a.bound + (int64_t)blockIdx.x * a.bstride;
    const int ge = a.ge, goe = a.goe;
    __shared__ unsigned long long s_next;
    for (;;) {
        // fetch the next group: one atomic by lane 0, broadcast through LDS
        __syncthreads();
        if (lane == 0) s_next = atomicAdd(a.counter, 1ull);
        __syncthreads();
        const int64_t g = uniform64(s_next);
        if (g >= a.ngroups) break;
        int pid = -1;       // output slot (mode 0: pair id)
        int sid = -1;       // sequence of this lane
        const uint8_t *cen = a.center;
        int m = a.m;
        int cid = -1;
        if (a.mode == 0) {
            pid = a.order ? a.order[g * 64 + lane] : (g * 64 + lane < a.nseq ? (int)(g * 64 + lane) : -1);
            sid = pid;
        } else {
            int64_t apos = -1, b0;
            if (a.mode == 1) {
                tri_group(a.gtotal - 1 - (a.gfirst + g), a.nseq, 64, &apos, &b0);
                cid = a.perm[apos];
            } else {
                b0 = a.gb0[g];
                cid = a.gcen[g];
            }
            const int64_t bpos = b0 + lane;
            if (bpos < a.nseq && bpos > apos) {
                sid = a.perm[bpos];
                pid = (int)(g * 64 + lane);   // output slot (mode 2); a self pair scores 0
                if (sid == cid) sid = -1;
            }
            cen = a.res + a.off[cid];
            m = (int)(a.off[cid + 1] - a.off[cid]);
        }
        const int64_t so = sid >= 0 ? a.off[sid] : 0;
        const int n = sid >= 0 ? (int)(a.off[sid + 1] - so) : 0;
        const uint8_t *s = a.res + so;
        // prefetch base: the set's first residue for an empty lane (a group
        // that runs any column holds at least one residue)
        const uint8_t *sq = n > 0 ? s : a.res;
        int nmax = n;
        if (a.mode == 0 && a.gnmax) {
            nmax = a.gnmax[g];
        } else {
#pragma unroll
            for (int sh = 1; sh < 64; sh <<= 1) nmax = max(nmax, __shfl_xor(nmax, sh));
        }
        m = __builtin_amdgcn_readfirstlane(m);        // same in every lane
        nmax = __builtin_amdgcn_readfirstlane(nmax);  // same in every lane
        const int nstrips = (m + kT - 1) / kT;
        const int G = (nmax + 3) >> 2;
        uint32_t *cw = TB ? a.codes + a.gcode_base[g] + lane * 8 : nullptr;
        uint32_t *stage = stage_all + lane * 8;
        BestCell best{0, 0x7fffffff, 0x7fffffff};
        int hmax = 0;
        for (int st = 0; st < nstrips; ++st) {
            const int i0 = st * kT;
            __syncthreads();
            for (int x = lane; x < (kAlphaMax + 1) * kT; x += 64) {
                const int r = x / kT, t = x - r * kT;
                int v = kNegProf;
                if (r < a.alpha && i0 + t < m) v = (int)smat[(cen[i0 + t] & 31) * 32 + r] + goe;
                prof[r * kPS + t] = v;
            }
            __syncthreads();
            int hg[kT], e[kT];
#pragma unroll
            for (int t = 0; t < kT; ++t) { hg[t] = -goe; e[t] = 0; }
            int diag0 = -goe;
            // The first strip reads residues from the lane's sequence and
            // leaves each column's code in its boundary cell (bits 26-31 of
            // F*, which stays below 2^23 for lengths < 65536 and |scores| <
            // 128); later strips get residue and boundary in one load.  A
            // block of kB columns is fetched one block ahead into the other of
            // two buffers, so the load latency overlaps a block of cells.  The
            // loads are unconditional (indexes clamped into the lane's
            // sequence and the group's boundary row) and so is the boundary
            // store, which keeps the wait counts exact across blocks.  Every
            // block is whole: columns past nmax (up to nmaxp, a multiple of kB)
            // are padding columns as for a lane's columns past n, whose cells
            // stay below an earlier cell of the lane and never win the end cell.
            const int nlast = max(n - 1, 0);
            const int nmaxp = (nmax + kB - 1) / kB * kB;
            auto strip = [&](auto first_tag) {
                constexpr bool FIRST = decltype(first_tag)::value;
                auto fetch = [&](int j0, int2 (&bq)[kB]) {
#pragma unroll
                    for (int b = 0; b < kB; ++b) {
                        const int j = min(j0 + b, nmaxp);
                        if (FIRST) bq[b].x = (int)sq[min(j - 1, nlast)];
                        else bq[b] = load_agent(bnd + (int64_t)(j - 1) * 64 + lane);
                    }
                };
                auto block = [&](int j0, const int2 (&bc)[kB]) {
#pragma unroll
                    for (int b = 0; b < kB; ++b) {
                        const int j = j0 + b;
                        int upg, upf, r;
                        if (FIRST) {
                            upg = -goe;
                            upf = 0;
                            r = (j <= n) ? (bc[b].x & 31) : kPad;
                        } else {
                            upg = bc[b].x;
                            upf = bc[b].y & kFMask;
                            r = (int)((uint32_t)bc[b].y >> kFBits);
                        }
                        int diag = diag0;
                        diag0 = upg;
                        const int *prow = prof + r * kPS;
                        int p[kT];
#pragma unroll
                        for (int t = 0; t < kT; ++t) p[t] = prow[t];
                        uint32_t w0 = 0, w1 = 0;
                        int colkey = 0;
#pragma unroll
                        for (int t = 0; t < kT; t += 2) {
                            const int h0 = sw_cell<TB>(hg[t], e[t], diag, upg, upf, p[t], ge, goe,
                                                       t < 8 ? w0 : w1);
                            const int h1 = sw_cell<TB>(hg[t + 1], e[t + 1], diag, upg, upf, p[t + 1], ge, goe,
                                                       t < 8 ? w0 : w1);
                            if (ENDC) colkey = vmax3(colkey, (h0 << 5) | (31 - t), (h1 << 5) | (30 - t));
                            else hmax = vmax3(hmax, h0, h1);
                        }
                        bnd[(int64_t)(j - 1) * 64 + lane] = make_int2(upg, (int)((uint32_t)upf | (uint32_t)r << kFBits));
                        if (TB) {
                            stage[2 * b] = w0;
                            stage[2 * b + 1] = w1;
                            if (b == kB - 1) {
                                const uint4 lo = *reinterpret_cast<const uint4 *>(stage);
                                const uint4 hi = *reinterpret_cast<const uint4 *>(stage + 4);
                                uint4 *dst = reinterpret_cast<uint4 *>(cw + ((int64_t)st * G + ((j - 1) >> 2)) * 512);
                                dst[0] = lo;
                                dst[1] = hi;
                            }
                        }
                        if (ENDC) {
                            // later strips hold larger i: on equal H they win only with a smaller j
                            const int ch = colkey >> 5;
                            if (ch > 0 && (ch > best.h || (ch == best.h && j < best.j))) {
                                best.h = ch;
                                best.j = j;
                                best.i = i0 + (31 - (colkey & 31));
                            }
                        }
                    }
                };
                int2 bA[kB], bB[kB];
                fetch(1, bA);
                for (int j0 = 1; j0 <= nmaxp; j0 += 2 * kB) {
                    fetch(j0 + kB, bB);
                    block(j0, bA);
                    if (j0 + kB > nmaxp) break;
                    fetch(j0 + 2 * kB, bA);
                    block(j0 + kB, bB);
                }
            };
            if (nmax > 0) {
                if (st == 0) strip(std::true_type{});
                else strip(std::false_type{});
            }
        }
        if (ENDC) hmax = best.h;
        if (a.mode == 0) {
            if (pid >= 0) {
                a.score[pid] = hmax;
                if (ENDC && a.endcell) {
                    a.endcell[2 * pid] = best.h > 0 ? best.i + 1 : 0;
                    a.endcell[2 * pid + 1] = best.h > 0 ? best.j : 0;
                }
                if (ENDC && a.cells4)
                    a.cells4[pid] = make_int4(0, 0, best.h > 0 ? best.i + 1 : 0, best.h > 0 ? best.j : 0);
            }
        } else {
            const int v = sid >= 0 ? hmax : 0;
            if (a.score && pid >= 0) a.score[pid] = v;
            if (a.mode == 1 && sid >= 0) atomicAdd(reinterpret_cast<unsigned long long *>(a.sums + sid), (unsigned long long)v);
            int tot = v;
#pragma unroll
            for (int sh = 1; sh < 64; sh <<= 1) tot += __shfl_xor(tot, sh);
            if (lane == 0) {
                const int slot = a.mode == 1 ? cid : a.gslot[g];
                atomicAdd(reinterpret_cast<unsigned long long *>(a.sums + slot), (unsigned long long)(int64_t)tot);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Packed 16-bit score-only strip kernel (center selection: modes 1 and 2).
// Each lane scores one partner against two centers at once, the first
// center in the low and the second in the high half of every register, with
// v_pk_* 16-bit integer ops.  Both halves read the profile at the partner's residue, so one
// LDS row holds the two centers' scores side by side and is used as it
// comes (two partners per lane against one center took a v_perm_b32 per cell to
// put two rows together), and a group has 64 partners rather than 128.
//
// Rows 2k and 2k + 1 of a strip hold every value plus ge (k + 1) (and the bias):
// going down into an even row then costs F nothing, and E pays its ge after its
// maximum.  With H - go kept in hg,
//   E = max(E', hg', floor + ge) - ge;   F = max(F_up, hg_up) (- ge into an odd row);
//   H = max(hg_diag + P, E, F);          hg = H - go
// (' the previous column), which is six and a half packed ops per two cells, and
// half a maximum for the running maximum of each pair of rows (one register for
// both, as they share their offset; they meet at the group's end).  The last row gives
// 16 ge back at the strip's boundary.  F needs no floor: H has E's.
//
// A strip has 32 rows, at three wavefronts per SIMD: the boundaries of all groups
// in flight (1.1 GB) go through memory, and with 16 rows the kernel was bound by that
// (4.2 TB/s of a copy's 4.66).  Now VALU issue bounds it (238 instructions per
// column).  1,500 proteins of 150-600, all pairs: 31.3 ms with 16 rows, 8.5 ops and
// groups of 128 partners; 25.2 with 16 rows; 23.6 with four wavefronts per SIMD, which
// leaves 128 registers and spills around the loops; 22.4; 21.2 with the groups in order of
// cost.  The host uses this kernel only when
// every H plus go + ge plus 18 ge stays below 16000 and every H below 15000, so that no
// biased value leaves [0, 0x7c00) and a padding profile entry can never be a source.
//
// Strip boundaries per lane and column: packed hg and packed F (int2) and the
// residue code (a byte), written by every strip and read by the next one
// with agent-scope loads (as in the 32-bit kernel).
// ---------------------------------------------------------------------------
constexpr int kC = 2;         // columns per prefetch block
constexpr int kT2 = 32;       // rows of a strip
constexpr int kPS2 = kT2 + 4; // LDS row stride of the profile: residues spread over the banks

__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3)))
sw_inter16_kernel(InterArgs a) {
    __shared__ __attribute__((aligned(16))) uint32_t prof[(kAlphaMax + 1) * kPS2];   // [r][32] (first, second center)
    __shared__ int8_t smat[kAlphaMax * kAlphaMax];
    __shared__ unsigned long long s_next;
    const int lane = threadIdx.x;
    for (int x = lane; x < kAlphaMax * kAlphaMax; x += 64) {
        const int r = x >> 5, q = x & 31;
        smat[x] = (r < a.alpha && q < a.alpha) ? a.mat[r * a.alpha + q] : (int8_t)0;
    }
    // per workgroup: int2 (packed hg, packed F) per lane and column, then the
    // lane's residue code (a byte) per column
    int2 *bnd = reinterpret_cast<int2 *>(reinterpret_cast<uint8_t *>(a.bound) + (int64_t)blockIdx.x * a.bstride * 9);
    uint8_t *bres = reinterpret_cast<uint8_t *>(bnd + a.bstride);
    const uint32_t ulane = (uint32_t)lane;   // (unsigned: a scalar column address plus a lane offset)
    auto both = [](int v) __attribute__((always_inline)) { return pk16{(short)v, (short)v}; };
    const int go = a.goe - a.ge;
    const pk16 ge2 = both(a.ge), go2 = both(go), last2 = both(kT2 / 2 * a.ge);
    pk16 flo[kT2 / 2];   // the floor of each pair of rows, plus ge
#pragma unroll
    for (int k = 0; k < kT2 / 2; ++k) flo[k] = both(kBias16 + a.ge * (k + 2));
    const pk16 top2 = both(kBias16 - go);   // hg above the first row: no offset
    for (;;) {
        __syncthreads();
        if (lane == 0) s_next = atomicAdd(a.counter, 1ull);
        __syncthreads();
        const int64_t g = uniform64(s_next);
        if (g >= a.ngroups) break;
        int64_t p0 = -1, p1 = -1, b0;   // positions that a partner has to be above
        int c0, c1;
        if (a.mode == 1) {
            pair_group(a.gorder ? a.gorder[g] : a.gtotal - 1 - (a.gfirst + g), a.nseq, &p0, &b0);
            p1 = p0 + 1;
            c0 = a.perm[p0];
            c1 = a.perm[p1];
        } else {
            b0 = a.gb0[g];
            c0 = a.gcen[g];
            c1 = a.gcen2[g];   // -1: none
        }
        const int64_t pos = b0 + lane;
        int sid = pos < a.nseq && pos > p0 ? a.perm[pos] : -1;
        const bool ok0 = sid >= 0 && sid != c0, ok1 = sid >= 0 && c1 >= 0 && pos > p1 && sid != c1;   // a self pair scores 0
        if (!ok0 && !ok1) sid = -1;
        const uint8_t *cen0 = a.res + a.off[c0], *cen1 = a.res + a.off[max(c1, 0)];
        const int m0 = __builtin_amdgcn_readfirstlane((int)(a.off[c0 + 1] - a.off[c0]));
        const int m1 = c1 < 0 ? 0 : __builtin_amdgcn_readfirstlane((int)(a.off[c1 + 1] - a.off[c1]));
        const int64_t so = sid >= 0 ? a.off[sid] : 0;
        const int n = sid >= 0 ? (int)(a.off[sid + 1] - so) : 0;
        // prefetch base: the set's first residue for an empty lane (a group
        // that runs any column holds at least one residue)
        const uint8_t *sq = n > 0 ? a.res + so : a.res;
        int nmax = n;
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1) nmax = max(nmax, __shfl_xor(nmax, sh));
        nmax = __builtin_amdgcn_readfirstlane(nmax);
        const int nstrips = (max(m0, m1) + kT2 - 1) / kT2;
        const int nmaxp = (nmax + kC - 1) / kC * kC;
        const int nlast = max(n - 1, 0);
        pk16 hm[kT2 / 2];   // running maxima of the pairs of rows
#pragma unroll
        for (int k = 0; k < kT2 / 2; ++k) hm[k] = flo[k] - ge2;
        for (int st = 0; st < nstrips && nmax > 0; ++st) {
            const int i0 = st * kT2;
            __syncthreads();
            for (int x = lane; x < (kAlphaMax + 1) * kT2; x += 64) {
                const int r = x >> 5, t = x & 31;
                const int add = (t & 1) ? go : a.goe;   // (from hg of a row with one ge less above an even row)
                int v0 = kPadProf16, v1 = kPadProf16;
                if (r < a.alpha && i0 + t < m0) v0 = (int)smat[(cen0[i0 + t] & 31) * 32 + r] + add;
                if (r < a.alpha && i0 + t < m1) v1 = (int)smat[(cen1[i0 + t] & 31) * 32 + r] + add;
                prof[r * kPS2 + t] = (uint32_t)(v0 & 0xffff) | ((uint32_t)v1 << 16);
            }
            __syncthreads();
            pk16 hg[kT2], e[kT2];
#pragma unroll
            for (int t = 0; t < kT2; ++t) hg[t] = e[t] = flo[t / 2] - ge2 - go2;
            pk16 diag0 = top2;
            auto strip = [&](auto first_tag) {
                constexpr bool FIRST = decltype(first_tag)::value;
                auto fetch = [&](int j0, int4 (&bq)[kC]) __attribute__((always_inline)) {
#pragma unroll
                    for (int b = 0; b < kC; ++b) {
                        const int j = min(j0 + b, nmaxp);
                        if (FIRST) {
                            bq[b].x = (int)sq[min(j - 1, nlast)];
                        } else {
                            const uint32_t at = __builtin_amdgcn_readfirstlane((j - 1) * 64);
                            const int2 v = load_agent(bnd + at + ulane);
                            const uint32_t rw = __hip_atomic_load(
                                reinterpret_cast<const uint32_t *>(bres + at + (ulane & ~3u)),
                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            bq[b] = make_int4(v.x, v.y, (int)(rw >> (8 * (lane & 3))) & 255, 0);
                        }
                    }
                };
                // two columns, the second a row behind the first: two chains of
                // dependent ops side by side
                auto block = [&](int j0, const int4 (&bc)[kC]) __attribute__((always_inline)) {
                    pk16 upg[kC], upf[kC], diag[kC], heven[kC];
                    int r[kC];
                    const uint4 *p4[kC];
                    uint4 w[kC];
#pragma unroll
                    for (int b = 0; b < kC; ++b) {
                        if (FIRST) {
                            upg[b] = top2;
                            upf[b] = top2;
                            r[b] = (j0 + b <= n) ? (bc[b].x & 31) : kPad;
                        } else {
                            upg[b] = as_pk((uint32_t)bc[b].x);
                            upf[b] = as_pk((uint32_t)bc[b].y);
                            r[b] = bc[b].z;
                        }
                        diag[b] = diag0;
                        diag0 = upg[b];
                        p4[b] = reinterpret_cast<const uint4 *>(prof + r[b] * kPS2);
                    }
#pragma unroll
                    for (int s = 0; s <= kT2; ++s) {
#pragma unroll
                        for (int b = 0; b < kC; ++b) {
                            const int t = s - b;
                            if (t < 0 || t >= kT2) continue;
                            if ((t & 3) == 0) w[b] = p4[b][t >> 2];
                            const uint32_t p = (t & 3) == 0 ? w[b].x : (t & 3) == 1 ? w[b].y : (t & 3) == 2 ? w[b].z : w[b].w;
                            const pk16 en = max3h(e[t], hg[t], flo[t / 2]) - ge2;
                            const pk16 fn = (t & 1) ? pmax(upf[b], upg[b]) - ge2 : pmax(upf[b], upg[b]);
                            const pk16 hh = max3h(diag[b] + as_pk(p), en, fn);
                            if (t & 1) hm[t / 2] = max3h(hm[t / 2], heven[b], hh);
                            else heven[b] = hh;
                            diag[b] = hg[t];
                            hg[t] = hh - go2;
                            e[t] = en;
                            upg[b] = hg[t];
                            upf[b] = fn;
                        }
                    }
#pragma unroll
                    for (int b = 0; b < kC; ++b) {
                        const uint32_t at = __builtin_amdgcn_readfirstlane((j0 + b - 1) * 64);
                        (bnd + at)[ulane] = make_int2((int)as_u(upg[b] - last2), (int)as_u(upf[b] - last2));
                        (bres + at)[ulane] = (uint8_t)r[b];
                    }
                };
                int4 bA[kC], bB[kC];
                fetch(1, bA);
                for (int j0 = 1; j0 <= nmaxp; j0 += 2 * kC) {
                    fetch(j0 + kC, bB);
                    block(j0, bA);
                    if (j0 + kC > nmaxp) break;
                    fetch(j0 + 2 * kC, bA);
                    block(j0 + kC, bB);
                }
            };
            if (st == 0) strip(std::true_type{});
            else strip(std::false_type{});
        }
        pk16 hmax = both(kBias16);
#pragma unroll
        for (int k = 0; k < kT2 / 2; ++k) hmax = pmax(hmax, hm[k] - (flo[k] - ge2 - both(kBias16)));
        const uint32_t hx = as_u(hmax);
        const int v0 = ok0 ? (int)(hx & 0xffff) - kBias16 : 0;
        const int v1 = ok1 ? (int)(hx >> 16) - kBias16 : 0;
        if (a.mode == 1 && sid >= 0)
            atomicAdd(reinterpret_cast<unsigned long long *>(a.sums + sid), (unsigned long long)(v0 + v1));
        int t0 = v0, t1 = v1;
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1) {
            t0 += __shfl_xor(t0, sh);
            t1 += __shfl_xor(t1, sh);
        }
        if (lane == 0) {
            const int s0 = a.mode == 1 ? c0 : a.gslot[g], s1 = a.mode == 1 ? c1 : a.gslot2[g];
            atomicAdd(reinterpret_cast<unsigned long long *>(a.sums + s0), (unsigned long long)(int64_t)t0);
            if (c1 >= 0) atomicAdd(reinterpret_cast<unsigned long long *>(a.sums + s1), (unsigned long long)(int64_t)t1);
        }
    }
}

}  // namespace hk

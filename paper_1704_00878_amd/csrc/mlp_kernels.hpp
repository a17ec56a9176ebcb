// Learned center proposer: 3-mer features, a BF16 MLP on MFMA (FP32
// accumulation), its backward, Adam, candidate scores and top-k.
//
// The paper picks the center as the sequence most similar to all others; the
// exhaustive search is O(N^2) SW alignments.  The proposer maps each
// sequence to an embedding e so that e_a . e_b approximates SW(a, b) / 100;
// u_i = e_i . (sum_j e_j - e_i) then approximates sum_j SW(i, j) / 100, and
// its top candidates are judged exactly.
//
// All reductions run in a fixed order (no float atomics), so every result is
// run-to-run deterministic.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hk {

constexpr int kFeat = 8000, kHid = 256, kEmb = 64;

__device__ __forceinline__ uint16_t f2bf(float f) {   // round to nearest even
    const uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// X[r][400a + 20b + c] = count of the 3-mer abc (all codes < 20) in sequence
// rows[r] (rows == null: r), as bf16 bits.  One workgroup per row, counts in LDS.
__global__ void __launch_bounds__(256)
featurize_kernel(const uint8_t *res, const int64_t *off, const int32_t *rows, int nrows, uint16_t *X) {
    __shared__ int cnt[kFeat];
    const int r = blockIdx.x;
    if (r >= nrows) return;
    const int k = rows ? rows[r] : r;
    const uint8_t *s = res + off[k];
    const int n = (int)(off[k + 1] - off[k]);
    for (int x = threadIdx.x; x < kFeat; x += 256) cnt[x] = 0;
    __syncthreads();
    for (int p = threadIdx.x; p + 2 < n; p += 256) {
        const int a = s[p], b = s[p + 1], c = s[p + 2];
        if (a < 20 && b < 20 && c < 20) atomicAdd(&cnt[400 * a + 20 * b + c], 1);
    }
    __syncthreads();
    uint16_t *row = X + (int64_t)r * kFeat;
    for (int x = threadIdx.x; x < kFeat / 8; x += 256) {
        uint32_t w[4];
#pragma unroll
        for (int y = 0; y < 4; ++y)
            w[y] = (uint32_t)f2bf((float)cnt[8 * x + 2 * y]) | ((uint32_t)f2bf((float)cnt[8 * x + 2 * y + 1]) << 16);
        reinterpret_cast<uint4 *>(row)[x] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

__global__ void iota_kernel(int32_t *p, int n) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x < n) p[x] = x;
}

__global__ void gather_f32_kernel(const float *src, const int32_t *idx, int n, float *dst) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x < n) dst[x] = src[idx[x]];
}

// Gather rows of a bf16 matrix: dst[r] = src[idx[r]] (width in elements).
__global__ void gather_rows_kernel(const uint16_t *src, const int32_t *idx, int nrows, int width, uint16_t *dst) {
    const int r = blockIdx.x;
    if (r >= nrows) return;
    const uint16_t *s = src + (int64_t)idx[r] * width;
    uint16_t *d = dst + (int64_t)r * width;
    for (int x = threadIdx.x; x < width; x += blockDim.x) d[x] = s[x];
}

// ---------------------------------------------------------------------------
// C[M x N] = op(A)[M x K] . op(B)[K x N] on v_mfma_f32_32x32x16_bf16.
//   op(A)(m, k) = TA ? A[k*lda + m] : A[m*lda + k]
//   op(B)(k, n) = TB ? B[n*ldb + k] : B[k*ldb + n]
// Workgroup tile 64 x 64, four waves of 32 x 32, K staged through LDS in 32s
// (k contiguous for both operands).  Epilogues:
//   0: C = acc (+ bias[n])
//   1: C = acc + bias[n] (pre-activation), Hb = bf16(relu(C))
//   2: D = acc * (Hpre > 0) (relu backward), Db = bf16(D)
//   3: as 2, Db packed (pack_index; rows up to the next 64 as zeros)
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

struct GemmArgs {
    const uint16_t *A;
    const uint16_t *B;
    int M, N, K, lda, ldb;
    float *C;
    int ldc;
    const float *bias;
    uint16_t *Cb;          // bf16 output (epilogues 1, 2)
    int ldcb;
    const float *Hpre;     // epilogue 2 mask source
    int ldh;
};

constexpr int kBK = 32, kLdsK = kBK + 8;

// epilogue EPI of element (gm, gn)
template <int EPI>
__device__ __forceinline__ void gemm_out(const GemmArgs &g, int gm, int gn, float v) {
    if (EPI == 0) {
        if (g.bias) v += g.bias[gn];
        g.C[(int64_t)gm * g.ldc + gn] = v;
    } else if (EPI == 1) {
        v += g.bias ? g.bias[gn] : 0.f;
        if (g.C) g.C[(int64_t)gm * g.ldc + gn] = v;
        g.Cb[(int64_t)gm * g.ldcb + gn] = f2bf(v > 0.f ? v : 0.f);
    } else {
        const float z = g.Hpre[(int64_t)gm * g.ldh + gn];
        const float d = z > 0.f ? v : 0.f;
        g.C[(int64_t)gm * g.ldc + gn] = d;
        g.Cb[(int64_t)gm * g.ldcb + gn] = f2bf(d);
    }
}

template <bool TA, bool TB, int EPI>
__global__ void __launch_bounds__(256)
gemm_bf16_kernel(GemmArgs g) {
    __shared__ uint16_t As[64][kLdsK];
    __shared__ uint16_t Bs[64][kLdsK];
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    f32x16_t acc;
#pragma unroll
    for (int x = 0; x < 16; ++x) acc[x] = 0.f;
    for (int k0 = 0; k0 < g.K; k0 += kBK) {
        // stage A (64 x 32) and B (32 x 64): 8 elements per thread each
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int q = tid * 8 + e;           // 0 .. 2047
            int mm, kk;
            if (TA) { kk = q >> 6; mm = q & 63; }   // consecutive threads walk m (contiguous in memory)
            else { mm = q >> 5; kk = q & 31; }      // consecutive threads walk k
            const int gm = m0 + mm, gk = k0 + kk;
            uint16_t v = 0;
            if (gm < g.M && gk < g.K) v = TA ? g.A[(int64_t)gk * g.lda + gm] : g.A[(int64_t)gm * g.lda + gk];
            As[mm][kk] = v;
            int nn;
            if (TB) { nn = q >> 5; kk = q & 31; }
            else { kk = q >> 6; nn = q & 63; }
            const int gn = n0 + nn, gk2 = k0 + kk;
            uint16_t w = 0;
            if (gn < g.N && gk2 < g.K) w = TB ? g.B[(int64_t)gn * g.ldb + gk2] : g.B[(int64_t)gk2 * g.ldb + gn];
            Bs[nn][kk] = w;
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < kBK; ks += 16) {
            const int kk = ks + 8 * (lane >> 5);
            const uint4 av = *reinterpret_cast<const uint4 *>(&As[wm + (lane & 31)][kk]);
            const uint4 bv = *reinterpret_cast<const uint4 *>(&Bs[wn + (lane & 31)][kk]);
            bf16x8_t a8, b8;
            __builtin_memcpy(&a8, &av, 16);
            __builtin_memcpy(&b8, &bv, 16);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a8, b8, acc, 0, 0, 0);
        }
        __syncthreads();
    }
    // acc[x]: row (x/4)*8 + (lane/32)*4 + x%4, column lane%32 of the wave tile
    const int gn = n0 + wn + (lane & 31);
    if (gn >= g.N) return;
#pragma unroll
    for (int x = 0; x < 16; ++x) {
        const int gm = m0 + wm + (x >> 2) * 8 + (lane >> 5) * 4 + (x & 3);
        if (gm >= g.M) continue;
        gemm_out<EPI>(g, gm, gn, acc[x]);
    }
}

// ---------------------------------------------------------------------------
// The same product from a packed B and an A of 16-byte rows, pipelined.
//
// The 64 x 64 kernel above loads two bytes at a time and waits for each 32-deep
// slice: X . W1 ran at 5% of the copy rate.  Here B is laid out beforehand as
// the fragments the matrix instruction takes (pack_index), so each wavefront
// loads its own columns' fragments straight into registers, PF slices of 64 k
// ahead; A goes through two LDS buffers with one barrier per slice, loaded 16
// bytes a thread (or 8 k-rows of CW elements, turned with v_perm, where k is
// the slow index), also PF slices ahead.  LDS holds octets of k as planes of
// 16-byte slots, one per row, so a fragment read touches consecutive slots;
// planes are padded so that the writes of one instruction start on different
// banks too.  X . W1 went 480 -> 22 us at 2,048 rows (a serial chain of 500
// matrix instructions, 32 cycles each at least, and their fragments from L2) and
// 1400 -> 100-112 us at 16,384 (262 MB of X, 2.4 TB/s); X^T . dZ 141 -> 18 us at
// 2,048 rows; staging B through LDS as well took 35 / 125 / 25.  The accumulation runs over k in the same order with the same
// instruction as above, so the results are the same bits.
// ---------------------------------------------------------------------------
// Packed operand: element (k, n) of a K x N matrix (N a multiple of 32, K
// rounded up to 64 with zeros) sits at the lane and half where
// v_mfma_f32_32x32x16_bf16 wants it; a fragment (16 k x 32 n) is 1 KiB.
__host__ __device__ __forceinline__ int64_t pack_index(int k, int n, int N) {
    return ((int64_t)(k >> 4) * (N >> 5) + (n >> 5)) * 512 + ((n & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
}

// dst = packed K x N of src (T: element (k, n) at src[n * ld + k], else at
// src[k * ld + n]).  One thread per 8 k of a column.
template <bool T>
__device__ __forceinline__ void pack_octet(const uint16_t *src, int ld, int K, int N, uint16_t *dst, int x) {
    const int n = x % N, k0 = x / N * 8;
    uint16_t h[8];
#pragma unroll
    for (int y = 0; y < 8; ++y)
        h[y] = k0 + y < K ? (T ? src[(int64_t)n * ld + k0 + y] : src[(int64_t)(k0 + y) * ld + n]) : (uint16_t)0;
    uint4 v;
    __builtin_memcpy(&v, h, 16);
    *reinterpret_cast<uint4 *>(dst + pack_index(k0, n, N)) = v;
}
__host__ __device__ __forceinline__ int pack_octets(int K, int N) { return (K + 63) / 64 * 8 * N; }

constexpr int kGK = 64;   // k per slice

template <int V> struct GVec;
template <> struct GVec<2> { typedef uint32_t T; };
template <> struct GVec<4> { typedef uint2 T; };
template <> struct GVec<8> { typedef uint4 T; };

// One operand's tile of ROWS rows x kGK k.  T: k is the slow index in memory
// (element (row, k) at p[k * ld + row]); else p[row * ld + k].
template <int ROWS, bool T, int THREADS>
struct GTile {
    static constexpr int PER = ROWS * kGK / THREADS;            // elements per thread
    static constexpr int CW = T ? PER / 8 : 8;                  // contiguous elements per load
    static constexpr int NL = T ? 8 : PER / 8;                  // loads per thread
    static constexpr int SPAN = T ? ROWS / CW : ROWS;           // slots of a sub-plane
    static constexpr int PAD = T ? 8 / CW : 1;
    static constexpr int PLANE = T ? CW * (SPAN + PAD) : ROWS + PAD;   // slots per octet
    static constexpr int BYTES = 8 * PLANE * 16;
    typedef typename GVec<CW>::T V;
    static_assert(PER % 8 == 0 && (!T || CW == 2 || CW == 4 || CW == 8), "tile split");
    static_assert(T ? (8 * (ROWS / CW) == THREADS) : (ROWS * 8 == THREADS * NL), "tile split");

    static __device__ __forceinline__ int slot(int r) { return T ? (r % CW) * (SPAN + PAD) + r / CW : r; }

    // This thread's first element of a slice (k from 0): rows beyond the last
    // one are read as the last one (their products are not written out), so
    // the loads of a full slice need no test.
    struct Src {
        const uint16_t *p[T ? 1 : NL];
        int64_t ld;
    };
    static __device__ __forceinline__ Src src(const uint16_t *p, int64_t ld, int r0, int rows) {
        const int t = threadIdx.x;
        Src q;
        q.ld = ld;
        if constexpr (T) {
            q.p[0] = p + (int64_t)(8 * (t / SPAN)) * ld + min(r0 + (t % SPAN) * CW, rows - CW);
        } else {
#pragma unroll
            for (int x = 0; x < NL; ++x)
                q.p[x] = p + (int64_t)min(r0 + (t >> 3) + x * (THREADS / 8), rows - 1) * ld + 8 * (t & 7);
        }
        return q;
    }
    // the slice of k from k0, all of it inside K
    static __device__ __forceinline__ void load(const Src &q, int k0, V *v) {
        if constexpr (T) {
            const uint16_t *p = q.p[0] + k0 * q.ld;
#pragma unroll
            for (int x = 0; x < 8; ++x) v[x] = *reinterpret_cast<const V *>(p + x * q.ld);
        } else {
#pragma unroll
            for (int x = 0; x < NL; ++x) v[x] = *reinterpret_cast<const V *>(q.p[x] + k0);
        }
    }
    // the last slice of a K that is no multiple of the slice: zeros beyond K
    static __device__ __forceinline__ void load_tail(const Src &q, int k0, int K, V *v) {
        const int t = threadIdx.x;
        if constexpr (T) {
            const int k = k0 + 8 * (t / SPAN);
            const uint16_t *p = q.p[0] + k0 * q.ld;
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                v[x] = V{};
                if (k + x < K) v[x] = *reinterpret_cast<const V *>(p + x * q.ld);
            }
        } else {
#pragma unroll
            for (int x = 0; x < NL; ++x) {
                v[x] = V{};
                if (k0 + 8 * (t & 7) < K) v[x] = *reinterpret_cast<const V *>(q.p[x] + k0);
            }
        }
    }

    static __device__ __forceinline__ void store(uint4 *lds, const V *v) {
        const int t = threadIdx.x;
        if constexpr (T) {
            const int c = t % SPAN, o = t / SPAN;
            uint32_t w[8][CW / 2];
#pragma unroll
            for (int x = 0; x < 8; ++x) __builtin_memcpy(w[x], &v[x], 2 * CW);
#pragma unroll
            for (int j = 0; j < CW; ++j) {
                uint32_t d[4];
                // halves j of eight k-rows, in pairs (low half of the first operand last in v_perm's numbering)
#pragma unroll
                for (int y = 0; y < 4; ++y)
                    d[y] = __builtin_amdgcn_perm(w[2 * y + 1][j / 2], w[2 * y][j / 2],
                                                 (j & 1) ? 0x07060302u : 0x05040100u);
                lds[o * PLANE + j * (SPAN + PAD) + c] = make_uint4(d[0], d[1], d[2], d[3]);
            }
        } else {
            const int o = t & 7;
#pragma unroll
            for (int x = 0; x < NL; ++x) lds[o * PLANE + (t >> 3) + x * (THREADS / 8)] = v[x];
        }
    }
};

// BM x BN per workgroup, WM x WN per wavefront, PF slices in flight.  A's k is
// its slow index when TA (as op(A) above); g.B is packed.
template <int BM, int BN, int WM, int WN, bool TA, int EPI, int PF>
__global__ void __launch_bounds__(64 * (BM / WM) * (BN / WN))
gemm_tile_kernel(GemmArgs g, int mtiles, int ntiles) {
    constexpr int THREADS = 64 * (BM / WM) * (BN / WN);
    constexpr int RM = WM / 32, RN = WN / 32, KS = kGK / 16;
    static_assert(PF % 2 == 0 && KS == 4, "two LDS buffers, four multiplies per slice");
    typedef GTile<BM, TA, THREADS> TAt;
    __shared__ uint4 gsm[2][8 * TAt::PLANE];
    // the column tiles of a row tile run on one XCD (blocks go round the 8
    // XCDs), which reads the rows into its L2 once
    const int xcd = blockIdx.x & 7, bs = blockIdx.x >> 3;
    const int mt = xcd + 8 * (bs / ntiles), nt = bs % ntiles;
    if (mt >= mtiles) return;
    const int m0 = mt * BM, n0 = nt * BN;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wm = (wave / (BN / WN)) * WM, wn = (wave % (BN / WN)) * WN;
    f32x16_t acc[RM][RN];
#pragma unroll
    for (int a = 0; a < RM; ++a)
#pragma unroll
        for (int b = 0; b < RN; ++b)
#pragma unroll
            for (int x = 0; x < 16; ++x) acc[a][b][x] = 0.f;
    typename TAt::V va[PF][TAt::NL];
    bf16x8_t fa[2][KS][RM], fb[PF][KS][RN];
    const typename TAt::Src ga = TAt::src(g.A, g.lda, m0, g.M);
    const int nf = g.K / kGK;                       // full slices
    const int slast = max(nf - 1, 0);
    const uint4 *gb = reinterpret_cast<const uint4 *>(g.B) + (int64_t)((n0 + wn) >> 5) * 64;
    const int kstride = (g.N >> 5) * 64;            // 16-byte units per 16 k
    int sa[RM];
#pragma unroll
    for (int a = 0; a < RM; ++a) sa[a] = TAt::slot(wm + 32 * a + (lane & 31)) + (lane >> 5) * TAt::PLANE;
    // the barrier orders LDS only: the register loads stay in flight across it
    auto sync = []() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    auto frags = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int a = 0; a < RM; ++a)
                __builtin_memcpy(&fa[buf][ks][a], &gsm[buf][sa[a] + 2 * ks * TAt::PLANE], 16);
    };
    auto getb = [&](int s, int p, int ks) __attribute__((always_inline)) {
        const uint4 *q = gb + (int64_t)(s * KS + ks) * kstride;
#pragma unroll
        for (int b = 0; b < RN; ++b) __builtin_memcpy(&fb[p][ks][b], q + b * 64 + lane, 16);
    };
    auto mfma = [&](int f, int p, int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < RM; ++a)
#pragma unroll
            for (int b = 0; b < RN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[f][ks][a], fb[p][ks][b], acc[a][b], 0, 0, 0);
    };
    if (nf > 0) {
        // slice x of A waits in va[x % PF], of B in fb[x % PF]; slices beyond
        // the last are read as the last (never multiplied)
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            TAt::load(ga, min(p, slast) * kGK, va[p]);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) getb(min(p, slast), p, ks);
        }
        TAt::store(gsm[0], va[0]);
        TAt::load(ga, min(PF, slast) * kGK, va[0]);
        sync();
        frags(0);
        TAt::store(gsm[1], va[1]);
        TAt::load(ga, min(PF + 1, slast) * kGK, va[1]);
        sync();
        // While slice s is multiplied from registers, A's fragments of slice
        // s + 1 are read, its slice s + 2 goes to the LDS buffer that slice s
        // was read from, and slices s + PF of B and s + 2 + PF of A are
        // requested: nothing waits inside the step but the barrier.
        auto step = [&](int s, int p) __attribute__((always_inline)) {
            const int q = (p + 2) % PF, sb = min(s + PF, slast);
            frags((p + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            mfma(p & 1, p, 0);
            __builtin_amdgcn_sched_barrier(0);
            TAt::store(gsm[p & 1], va[q]);
            getb(sb, p, 0);
            __builtin_amdgcn_sched_barrier(0);
            mfma(p & 1, p, 1);
            __builtin_amdgcn_sched_barrier(0);
            TAt::load(ga, min(s + 2 + PF, slast) * kGK, va[q]);
            getb(sb, p, 1);
            __builtin_amdgcn_sched_barrier(0);
            mfma(p & 1, p, 2);
            __builtin_amdgcn_sched_barrier(0);
            getb(sb, p, 2);
            __builtin_amdgcn_sched_barrier(0);
            mfma(p & 1, p, 3);
            __builtin_amdgcn_sched_barrier(0);
            getb(sb, p, 3);
            sync();
        };
        int s = 0;
        for (; s + PF <= nf; s += PF) {
#pragma unroll
            for (int p = 0; p < PF; ++p) step(s + p, p);
        }
#pragma unroll
        for (int p = 0; p < PF - 1; ++p)
            if (s + p < nf) step(s + p, p);
    }
    if (g.K % kGK) {   // (the last step's barrier follows every read of the first buffer)
        TAt::load_tail(ga, nf * kGK, g.K, va[0]);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) getb(nf, 0, ks);
        sync();
        TAt::store(gsm[0], va[0]);
        sync();
        frags(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) mfma(0, 0, ks);
    }
#pragma unroll
    for (int b = 0; b < RN; ++b) {
        const int gn = n0 + wn + 32 * b + (lane & 31);
#pragma unroll
        for (int a = 0; a < RM; ++a) {
            const int gm0 = m0 + wm + 32 * a + (lane >> 5) * 4;   // rows gm0 + 8 * (x / 4) + x % 4
            if constexpr (EPI == 3) {
                const int mpad = (g.M + kGK - 1) / kGK * kGK;
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    uint32_t w[2] = {0, 0};
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const int gm = gm0 + 8 * y + x;
                        if (gm < g.M) {
                            const float z = g.Hpre[(int64_t)gm * g.ldh + gn];
                            const float d = z > 0.f ? acc[a][b][4 * y + x] : 0.f;
                            g.C[(int64_t)gm * g.ldc + gn] = d;
                            w[x >> 1] |= (uint32_t)f2bf(d) << (16 * (x & 1));
                        }
                    }
                    if (gm0 + 8 * y < mpad)
                        *reinterpret_cast<uint2 *>(g.Cb + pack_index(gm0 + 8 * y, gn, g.N)) = make_uint2(w[0], w[1]);
                }
            } else {
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const int gm = gm0 + 8 * (x >> 2) + (x & 3);
                    if (gm < g.M) gemm_out<EPI>(g, gm, gn, acc[a][b][x]);
                }
            }
        }
    }
}

// Weights of the forward packed in one launch: W1 (kFeat x kHid), W2 (kHid x kEmb).
constexpr int kPackW1 = (kFeat + 63) / 64 * 8 * kHid, kPackW2 = kHid / 8 * kEmb, kPackW2T = kEmb / 8 * kHid;   // octets
__global__ void __launch_bounds__(256) pack_weights_kernel(const uint16_t *W1, const uint16_t *W2, uint16_t *P1,
                                                           uint16_t *P2) {
    const int x = blockIdx.x * 256 + threadIdx.x;
    if (x < kPackW1) pack_octet<false>(W1, kHid, kFeat, kHid, P1, x);
    else if (x < kPackW1 + kPackW2) pack_octet<false>(W2, kEmb, kHid, kEmb, P2, x - kPackW1);
}

// Operands of the backward in one launch: dE (rows x kEmb, fp32) as bf16 row
// by row (A of dZ) and packed (B of dW2), and W2 transposed, packed (B of dZ).
// One thread per 8 rows of a column of dE; rows beyond the last are packed as
// zeros.
__global__ void __launch_bounds__(256) pack_backward_kernel(const float *dE, int rows, uint16_t *dEb, uint16_t *Pd,
                                                            const uint16_t *W2, uint16_t *P2t) {
    const int x = blockIdx.x * 256 + threadIdx.x, nd = pack_octets(rows, kEmb);
    if (x < nd) {
        const int n = x % kEmb, r0 = x / kEmb * 8;
        uint16_t h[8];
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            h[y] = 0;
            if (r0 + y < rows) {
                h[y] = f2bf(dE[(int64_t)(r0 + y) * kEmb + n]);
                dEb[(int64_t)(r0 + y) * kEmb + n] = h[y];
            }
        }
        uint4 v;
        __builtin_memcpy(&v, h, 16);
        *reinterpret_cast<uint4 *>(Pd + pack_index(r0, n, kEmb)) = v;
    } else if (x < nd + kPackW2T) {
        pack_octet<true>(W2, kEmb, kEmb, kHid, P2t, x - nd);
    }
}

// Column sums in a fixed order: partial sums over row blocks of 1024, each
// added row by row from 0, then the partials in block order.  A workgroup
// takes 64 columns of one block: all 1024 threads fetch 128 rows at a time (one
// tile ahead) into LDS, from which the first wavefront adds
// its column's rows in order.  With one thread fetching and adding each
// column's rows itself, 2048 x 256 took 233 us (one load in flight per
// add), and 16384 x 64 238; now 14 (with a 2048 x 64 beside it) and 13, bound by the
// serial chain of 1,024 adds.  Up to two matrices per launch (blocks x < c0 take
// the first).
constexpr int kColRows = 1024, kColTile = 128;
struct ColsumArgs {
    const float *A[2];
    int cols[2];      // multiples of 64
    float *part[2];   // [blocks][cols]
    float *out[2];
    int rows;
};
__global__ void __launch_bounds__(1024) colsum_partial_kernel(ColsumArgs a) {
    __shared__ float tile[2][kColTile][64];
    const int c0 = a.cols[0] / 64;
    const int w = (int)blockIdx.x >= c0 ? 1 : 0;
    const int cols = a.cols[w], col = ((int)blockIdx.x - w * c0) * 64;
    const int r0 = blockIdx.y * kColRows, rows = min(kColRows, a.rows - r0);
    const float *A = a.A[w] + (int64_t)r0 * cols + col;
    const int lane = threadIdx.x & 63, row = threadIdx.x >> 6;   // 16 rows at a time
    float v[kColTile / 16];
    auto get = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < kColTile / 16; ++x) {
            const int r = t * kColTile + 16 * x + row;
            v[x] = r < rows ? A[(int64_t)r * cols + lane] : 0.f;
        }
    };
    const int nt = (rows + kColTile - 1) / kColTile;
    float s = 0.f;
    get(0);
    for (int t = 0; t < nt; ++t) {
#pragma unroll
        for (int x = 0; x < kColTile / 16; ++x) tile[t & 1][16 * x + row][lane] = v[x];
        if (t + 1 < nt) get(t + 1);
        __syncthreads();   // the other tile was last read before the previous barrier
        if (row == 0) {
            const int n = min(kColTile, rows - t * kColTile);
            int r = 0;
            for (; r + 16 <= n; r += 16) {
                float q[16];
#pragma unroll
                for (int x = 0; x < 16; ++x) q[x] = tile[t & 1][r + x][lane];
#pragma unroll
                for (int x = 0; x < 16; ++x) s += q[x];
            }
            for (; r < n; ++r) s += tile[t & 1][r][lane];
        }
    }
    if (row == 0) a.part[w][(int64_t)blockIdx.y * cols + col + lane] = s;
}
__global__ void colsum_final_kernel(ColsumArgs a, int nblk) {
    int c = blockIdx.x * blockDim.x + threadIdx.x, w = 0;
    if (c >= a.cols[0]) {
        c -= a.cols[0];
        w = 1;
    }
    if (c >= a.cols[w]) return;
    float s = 0.f;
    for (int b = 0; b < nblk; ++b) s += a.part[w][(int64_t)b * a.cols[w] + c];
    a.out[w][c] = s;
}

// Pair loss: pairs (r, r + P).  dE (fp32); per-pair squared errors go to
// sq[P] for a fixed-order loss reduction.
// A workgroup takes 16 pairs: their rows go through LDS with coalesced loads,
// one thread per pair adds the products in order of d, and all threads write
// the gradients coalesced (with a thread per pair reading and writing its own
// rows, 1,024 pairs took 62 us; now 4).
constexpr int kLossPairs = 16;
__global__ void __launch_bounds__(256) pair_loss_kernel(const float *E, const float *target, int P, float *dE, float *sq) {
    __shared__ float ea[kLossPairs][kEmb + 1], eb[kLossPairs][kEmb + 1], gs[kLossPairs];
    const int p0 = blockIdx.x * kLossPairs, t = threadIdx.x;
    const int n = min(kLossPairs, P - p0);
    const float *A = E + (int64_t)p0 * kEmb, *B = E + (int64_t)(p0 + P) * kEmb;
#pragma unroll
    for (int x = t; x < kLossPairs * kEmb; x += 256)
        if (x / kEmb < n) {
            ea[x / kEmb][x % kEmb] = A[x];
            eb[x / kEmb][x % kEmb] = B[x];
        }
    __syncthreads();
    if (t < n) {
        float pred = 0.f;
#pragma unroll 16
        for (int d = 0; d < kEmb; ++d) pred += ea[t][d] * eb[t][d];
        const float diff = pred - target[p0 + t];
        sq[p0 + t] = diff * diff;
        gs[t] = 2.f * diff / (float)P;
    }
    __syncthreads();
    float *dA = dE + (int64_t)p0 * kEmb, *dB = dE + (int64_t)(p0 + P) * kEmb;
#pragma unroll
    for (int x = t; x < kLossPairs * kEmb; x += 256)
        if (x / kEmb < n) {
            dA[x] = gs[x / kEmb] * eb[x / kEmb][x % kEmb];
            dB[x] = gs[x / kEmb] * ea[x / kEmb][x % kEmb];
        }
}

// out[0] = sum(v[0..n)) / n in a fixed order (one workgroup).
__global__ void __launch_bounds__(256) mean_kernel(const float *v, int n, float *out) {
    __shared__ float part[256];
    float s = 0.f;
    const int per = (n + 255) / 256;
    const int lo = min(n, (int)threadIdx.x * per), hi = min(n, lo + per);
    for (int x = lo; x < hi; ++x) s += v[x];
    part[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int x = 0; x < 256; ++x) t += part[x];
        out[0] = n > 0 ? t / (float)n : 0.f;
    }
}

// Pair loss with a per-group term: groups of K consecutive pairs (K <= 64,
// one wavefront per group), loss = mean(diff^2) + lam * mean over groups of
// (mean diff of the group)^2.  dpred = 2 diff / P + 2 lam gmean / (G K).
__global__ void __launch_bounds__(64) pair_group_loss_kernel(const float *E, const float *target, int P, int K,
                                                             float lam, float *dE, float *sq, float *gsq) {
    const int g = blockIdx.x, l = threadIdx.x;
    const int G = P / K;
    const int r = g * K + l;
    float diff = 0.f, pred = 0.f;
    const float *a = E + (int64_t)r * kEmb, *b = E + (int64_t)(r + P) * kEmb;
    if (l < K) {
        for (int d = 0; d < kEmb; ++d) pred += a[d] * b[d];
        diff = pred - target[r];
        sq[r] = diff * diff;
    }
    float sum = diff;   // fixed-order tree over the wavefront
    for (int sh = 32; sh > 0; sh >>= 1) sum += __shfl_xor(sum, sh);
    const float gm = sum / (float)K;
    if (l == 0) gsq[g] = gm * gm;
    if (l >= K) return;
    const float gsc = 2.f * diff / (float)P + 2.f * lam * gm / ((float)G * (float)K);
    float *da = dE + (int64_t)r * kEmb, *db = dE + (int64_t)(r + P) * kEmb;
    for (int d = 0; d < kEmb; ++d) {
        da[d] = gsc * b[d];
        db[d] = gsc * a[d];
    }
}

// out[0] = mean(v[0..n)) + lam * mean(w[0..m)), each sum in a fixed order.
__global__ void __launch_bounds__(256) mean2_kernel(const float *v, int n, const float *w, int m, float lam,
                                                    float *out) {
    __shared__ float part[256];
    float res = 0.f;
    for (int which = 0; which < 2; ++which) {
        const float *x = which ? w : v;
        const int c = which ? m : n;
        float s = 0.f;
        const int per = (c + 255) / 256;
        const int lo = min(c, (int)threadIdx.x * per), hi = min(c, lo + per);
        for (int q = lo; q < hi; ++q) s += x[q];
        part[threadIdx.x] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.f;
            for (int q = 0; q < 256; ++q) t += part[q];
            res += (which ? lam : 1.f) * (c > 0 ? t / (float)c : 0.f);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = res;
}

// Adam with bias correction on fp32 masters; optional bf16 copy.
__global__ void adam_kernel(float *p, const float *gr, float *m, float *v, uint16_t *pb, int64_t n, float lr,
                            float b1, float b2, float eps, float c1, float c2) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x) {
        const float gx = gr[x];
        const float mx = b1 * m[x] + (1.f - b1) * gx;
        const float vx = b2 * v[x] + (1.f - b2) * gx * gx;
        m[x] = mx;
        v[x] = vx;
        const float mh = mx / c1, vh = vx / c2;
        const float px = p[x] - lr * mh / (sqrtf(vh) + eps);
        p[x] = px;
        if (pb) pb[x] = f2bf(px);
    }
}

// exponential moving average of parameters: e = d * e + (1 - d) * p
__global__ void ema_kernel(const float *p, float *e, int64_t n, float d) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x)
        e[x] = d * e[x] + (1.f - d) * p[x];
}

__global__ void f32_to_bf16_kernel(const float *src, uint16_t *dst, int64_t n) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x)
        dst[x] = f2bf(src[x]);
}

// targets: t[q] = score[q] / 100
__global__ void scale_targets_kernel(const int32_t *score, int n, float *t) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) t[q] = (float)score[q] / 100.f;
}

// u_i = e_i . (S - e_i) with S = sum_j e_j
__global__ void center_score_kernel(const float *E, const float *S, int n, float *u) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float *e = E + (int64_t)i * kEmb;
    float a = 0.f, b = 0.f;
    for (int d = 0; d < kEmb; ++d) { a += e[d] * S[d]; b += e[d] * e[d]; }
    const float r = a - b;
    u[i] = (r == r) ? r : -3.0e38f;   // NaN sorts last
}

// Top-k (largest first, ties to the lower index) by k rounds of block argmax.
// Pass 1: each workgroup reduces `chunk` entries of (val, idx) to its top k;
// pass 2 runs the same kernel over the partial results.
// A thread keeps its 16 entries in registers as 64-bit keys (the value's
// order-preserving bits, then the index complemented), so a round is a maximum
// over the wavefront's shuffles, one barrier, and a rescan by the one thread
// whose entry was taken.  Scanning all entries in LDS each round and reducing
// through eight barriers took 55 + 36 us for the two passes over 16,384 rows
// at k = 16; now 18 + 14 (a serial chain of k rounds).
constexpr int kTopkChunk = 4096;
constexpr float kTopkNone = -3.4e38f;   // values below it (or NaN) are never taken
__device__ __forceinline__ uint64_t topk_key(float v, int i) {
    if (!(v >= kTopkNone) || i == 0x7fffffff) return 0;
    const uint32_t b = __float_as_uint(v + 0.f);   // -0 ranks with +0
    return (uint64_t)(b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u)) << 32 | (uint32_t)~i;
}
__global__ void __launch_bounds__(256)
topk_kernel(const float *val, const int32_t *idx, int n, int k, float *oval, int32_t *oidx) {
    __shared__ uint64_t wmax[2][4];
    const int base = blockIdx.x * kTopkChunk;
    const int cnt = min(kTopkChunk, n - base);
    uint64_t key[kTopkChunk / 256], best = 0;
#pragma unroll
    for (int y = 0; y < kTopkChunk / 256; ++y) {
        const int x = y * 256 + threadIdx.x;
        key[y] = x < cnt ? topk_key(val[base + x], idx ? idx[base + x] : base + x) : 0;
        best = max(best, key[y]);
    }
    for (int r = 0; r < k; ++r) {
        uint64_t m = best;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t lo = __shfl_xor((int)(uint32_t)m, d), hi = __shfl_xor((int)(uint32_t)(m >> 32), d);
            m = max(m, (uint64_t)hi << 32 | lo);
        }
        uint64_t *w = wmax[r & 1];   // the other set was last read before the previous barrier
        if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = m;
        __syncthreads();
        m = max(max(w[0], w[1]), max(w[2], w[3]));
        if (threadIdx.x == 0) {
            const uint32_t b = (uint32_t)(m >> 32);
            oval[blockIdx.x * k + r] = m ? __uint_as_float(b ^ ((b >> 31) ? 0x80000000u : 0xffffffffu)) : kTopkNone;
            oidx[blockIdx.x * k + r] = m ? (int)~(uint32_t)m : 0x7fffffff;
        }
        if (m && best == m) {   // taken (keys are distinct)
            best = 0;
#pragma unroll
            for (int y = 0; y < kTopkChunk / 256; ++y) {
                if (key[y] == m) key[y] = 0;
                best = max(best, key[y]);
            }
        }
    }
}

}  // namespace hk

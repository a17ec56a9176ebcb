// Host runtime and C ABI of the center-star MSA library (gfx950).
//
// The runtime owns device scratch (traceback codes, boundary rows, plans) in
// a halign_ctx, plans each batch -- on the device from 2,048 pairs where its rule
// fits (plan_kernels.hpp), else on the host (length sort, grouping, chunking under a
// workspace cap) -- and launches the kernels on the caller's stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <fstream>
#include <initializer_list>
#include <functional>
#include <map>
#include <sstream>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <array>
#include <chrono>
#include <mutex>
#include <numeric>
#include <string>
#include <vector>

#include "../../include/halign.h"
#include "launch.hpp"
#include "msa_kernels.hpp"
#include "plan_kernels.hpp"
#include "strip_kernels.hpp"
#include "walk_kernels.hpp"
#include "nuc_kernels.hpp"
#include "nj_kernels.hpp"
#include "mlp_kernels.hpp"

namespace {

// message of the last failure on this thread (a fixed buffer: reporting an
// error allocates nothing)
thread_local char g_err[512];

int fail(int code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

#define HCHK(expr)                                                                   \
    do {                                                                             \
        hipError_t e_ = (expr);                                                      \
        if (e_ != hipSuccess)                                                        \
            return fail(HALIGN_E_DEVICE, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

using hk::launch_stream;
using hk::launch_stream16;
using hk::stream16_supported;
using hk::stream_supported;

#define RCHK(expr)                 \
    do {                           \
        int r_ = (expr);           \
        if (r_ != HALIGN_OK) return r_; \
    } while (0)

struct DevBuf {
    void *p = nullptr;
    size_t cap = 0;
};

struct HostBuf {
    void *p = nullptr;
    void *dev = nullptr;   // the device's address of p (the stage)
    size_t cap = 0;
};

}  // namespace

struct halign_ctx {
    int device = 0;
    bool counted = false;    // counted among its device's contexts (eval_contexts)
    size_t cap = 0;          // workspace cap for codes + boundary rows (0 = none)
    int num_cu = 256;
    size_t lds_max = 65536;
    size_t lds_cu = 65536;      // LDS of a CU: what one workgroup may take with the attribute set
    int last_pk = 0;          // the last batch ran the packed 16-bit wavefront kernel
    // device scratch
    DevBuf codes, bound, plan, counter, pairbuf, msabuf, spbuf, sbuf, histbuf;
    DevBuf mlp[10];          // learned-center scratch (features, activations, gradients, moments)
    // pinned host staging for plans: regions are taken in order within a
    // call (stage_off, plan_off) and never reused before the call ends, so the
    // copies of a captured graph each read their own region
    HostBuf stage;
    size_t stage_off = 0, plan_off = 0;
    hipEvent_t ev_stage = nullptr;
    bool stage_pending = false;
    bool stage_event = false;   // ev_stage was recorded after the pending copies
    // timing of the last call: one (start, forward end, walk end) event
    // triple per forward launch (chunk, route or graph replay)
    std::vector<std::array<hipEvent_t, 3>> tev;
    int ntev = 0;
    int64_t last_stats[4] = {0, 0, 0, 0};
    int fault_chunk = -1;    // test hook: chunk index whose first launch reports failure
    bool capturing = false;   // a hipGraph capture of halign_sw_batch is in progress
    int use_graph = 0;        // halign_msa passes HALIGN_GRAPH to its batch
    hipStream_t cap_stream = nullptr;
    hipStream_t aux_stream = nullptr;   // the tree's small joins beside the chip-wide ones
    struct GraphEntry {
        uint64_t key = 0;
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        DevBuf plan, codes, sbuf, bound, counter, pairbuf, spbuf;
        HostBuf stage;
    } gent;
    int64_t graph_launches = 0;
    int autotune = 0;         // 1: tune route / rows per lane / stream count per bucket
    int progress = 0;         // 1: a line on stderr after each chunk of a chunked batch
    std::array<int, 5> last_tune = {-1, 0, 1, 64, 0};
    std::map<std::string, std::array<int, 5>> tuned;   // bucket -> {route, R, stream multiplier, lanes per stream, packed}
    std::string tune_file;    // optional cache file (HALIGN_TUNE_CACHE)
    int *flag_host = nullptr; // pinned: (tag << 8 | largest residue code) of the last validated call
    int64_t *mail_host = nullptr, *mail_dev = nullptr;   // coherent pinned mailbox: width, sequence number, flag, five counts
    DevBuf nuctab, nucscr, nucdp;   // nucleotide path: segment table and matches, stretch lists, stretch scratch
    int64_t nuc_list = 0, nuc_rows = 0, nuc_codes = 0, nuc_big = 0;   // entries that nucscr and nucdp are laid out for
    int nuc_crowded[2] = {0, 0};    // k and segments of the last call whose matches outgrew the chain's LDS
    DevBuf rowck;                   // chunked rows: residues before each chunk of blocks, per row
    HostBuf njhost, njout;          // pinned: the tree's distances and the trees coming back
    DevBuf njF;                     // all rows' distances (sets where they are computed at once)
    hipEvent_t ev_nj = nullptr;     // the distances are in place (for aux_stream)
    DevBuf njrows, njD, njS, njacc, njB; // phylogeny: row lists and group tables, distance matrices, join scratch, slice counts, chip-wide join scratch
    int64_t mail_seq = 0;
    uint32_t vtag = 0;        // tag of the last eager code check
    uint32_t *vflag = nullptr;   // the flag word those tags were raised in (cleared when it changes)
    uint32_t check_tag = 0;   // tag validate_check expects (0 after a graph replay)
    int flag_alpha = 0;       // alphabet that value is checked against (0 = nothing pending)
    // HALIGN_HOST_TIMING=1: host time between labelled points of each
    // halign_msa call, one line on stderr per call
    int host_timing = 0;
    std::vector<std::pair<const char *, double>> hmarks;
    // learned center: pre-judge of the top prejudge_cand candidates by u
    // against prejudge_part common partners (0: off)
    int prejudge_cand = 0, prejudge_part = 0;
    // host planning scratch, kept between calls (no allocation per call)
    std::vector<int32_t> h_samp, h_pids, h_plen, h_cnt, h_sof, h_head, h_nxt, h_scount, h_cur, h_split;
    std::vector<int64_t> h_scols;
    // the last tuned-plan lookup, by its integer key
    int64_t tkey[4] = {-1, -1, -1, -1};
    std::array<int, 5> tval = {-1, 0, 1, 64, 0};
};

static void eval_contexts(int device, int change);

namespace {

void hmark(halign_ctx *ctx, const char *label) {
    if (!ctx->host_timing) return;
    const double us =
        std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now().time_since_epoch()).count();
    ctx->hmarks.push_back({label, us});
}

void hmark_print(halign_ctx *ctx) {
    if (!ctx->host_timing || ctx->hmarks.size() < 2) return;
    fprintf(stderr, "halign host us:");
    for (size_t q = 1; q < ctx->hmarks.size(); ++q)
        fprintf(stderr, " %s %.1f", ctx->hmarks[q].first, ctx->hmarks[q].second - ctx->hmarks[q - 1].second);
    fprintf(stderr, " (total %.1f)\n", ctx->hmarks.back().second - ctx->hmarks.front().second);
    ctx->hmarks.clear();
}

int grow(halign_ctx *ctx, DevBuf &b, size_t bytes) {
    if (bytes <= b.cap) return HALIGN_OK;
    size_t want = std::max(bytes, b.cap + b.cap / 2);
    want = (want + 4095) & ~size_t(4095);
    if (b.p) HCHK(hipFree(b.p));
    b.p = nullptr;
    b.cap = 0;
    if (hipMalloc(&b.p, want) != hipSuccess) {
        (void)hipGetLastError();
        b.p = nullptr;
        if (hipMalloc(&b.p, bytes) != hipSuccess) {
            (void)hipGetLastError();
            b.p = nullptr;
            return fail(HALIGN_E_NOMEM, "device allocation of %zu bytes failed", bytes);
        }
        want = bytes;
    }
    b.cap = want;
    (void)ctx;
    return HALIGN_OK;
}

// Pinned host memory kept between calls (nothing may be in flight to it).
int grow_host(HostBuf &b, size_t bytes) {
    if (bytes <= b.cap) return HALIGN_OK;
    if (b.p) HCHK(hipHostFree(b.p));
    b.p = nullptr;
    b.cap = 0;
    const size_t want = (bytes + bytes / 2 + 65535) & ~size_t(65535);
    HCHK(hipHostMalloc(&b.p, want, hipHostMallocDefault));
    b.cap = want;
    return HALIGN_OK;
}

// Event records are skipped while a graph is being captured (timing of a
// replay comes from events around the graph launch).
int record(halign_ctx *ctx, hipEvent_t e, hipStream_t st) {
    if (ctx->capturing) return HALIGN_OK;
    HCHK(hipEventRecord(e, st));
    return HALIGN_OK;
}

void free_buf(DevBuf &b) {
    if (b.p) (void)hipFree(b.p);
    b = DevBuf();
}

void graph_drop(halign_ctx *ctx) {
    auto &g = ctx->gent;
    if (g.exec) (void)hipGraphExecDestroy(g.exec);
    if (g.graph) (void)hipGraphDestroy(g.graph);
    for (DevBuf *b : {&g.plan, &g.codes, &g.sbuf, &g.bound, &g.counter, &g.pairbuf, &g.spbuf}) free_buf(*b);
    if (g.stage.p) (void)hipHostFree(g.stage.p);
    g = halign_ctx::GraphEntry();
}

// Copies from the pinned stage are in flight on a stream.  Calls that wait for
// their stream anyway clear stage_pending there; stage_close at a call's end
// records the event for the others (an event after every copy left a gap of 5 us
// before the forward kernel).
void stage_copied(halign_ctx *ctx) {
    if (ctx->capturing) return;
    ctx->stage_pending = true;
    ctx->stage_event = false;
}
int stage_close(halign_ctx *ctx, hipStream_t st) {
    if (ctx->stage_pending && !ctx->stage_event && !ctx->capturing) {
        HCHK(hipEventRecord(ctx->ev_stage, st));
        ctx->stage_event = true;
    }
    return HALIGN_OK;
}
int stage_wait(halign_ctx *ctx) {
    if (ctx->capturing) return HALIGN_OK;
    if (ctx->stage_pending) {
        if (ctx->stage_event) HCHK(hipEventSynchronize(ctx->ev_stage));
        else HCHK(hipDeviceSynchronize());   // a call that failed halfway, or regions regrown within one
        ctx->stage_pending = false;
    }
    return HALIGN_OK;
}

// Start of a call: the previous call's copies have left the pinned stage,
// whose regions are then taken from its start again; the timing triples
// restart too.
int stage_begin(halign_ctx *ctx) {
    RCHK(stage_wait(ctx));
    ctx->stage_off = 0;
    ctx->plan_off = 0;
    ctx->ntev = 0;
    return HALIGN_OK;
}

// `bytes` of the pinned stage, after the regions this call took already.
int stage_host(halign_ctx *ctx, size_t bytes, char **host) {
    const size_t o = (ctx->stage_off + 255) & ~size_t(255);
    if (o + bytes > ctx->stage.cap) {
        if (ctx->capturing) return fail(HALIGN_E_UNSUPPORTED, "plan staging outgrew its buffer under graph capture");
        RCHK(stage_wait(ctx));   // the regions taken so far have been copied
        if (ctx->stage.p) HCHK(hipHostFree(ctx->stage.p));
        ctx->stage.p = nullptr;
        ctx->stage.cap = 0;
        const size_t want = std::max<size_t>(2 * (o + bytes), 1 << 16);
        HCHK(hipHostMalloc(&ctx->stage.p, want, hipHostMallocDefault));
        ctx->stage.cap = want;
        if (hipHostGetDevicePointer(&ctx->stage.dev, ctx->stage.p, 0) != hipSuccess) ctx->stage.dev = nullptr;
    }
    *host = (char *)ctx->stage.p + o;
    ctx->stage_off = o + bytes;
    return HALIGN_OK;
}

// What a kernel reads a region of the stage by (nullptr: not mapped).
void *stage_dev(const halign_ctx *ctx, const char *host) {
    return ctx->stage.dev ? (char *)ctx->stage.dev + (host - (char *)ctx->stage.p) : nullptr;
}

// `bytes` of the device plan buffer, after the regions this call took already
// (a larger buffer replaces it only once the stream has drained).
int plan_dev(halign_ctx *ctx, size_t bytes, hipStream_t st, char **dev) {
    const size_t o = (ctx->plan_off + 255) & ~size_t(255);
    if (o + bytes > ctx->plan.cap) {
        if (ctx->capturing) return fail(HALIGN_E_UNSUPPORTED, "plan outgrew its buffer under graph capture");
        if (ctx->plan.p) HCHK(hipStreamSynchronize(st));
        RCHK(grow(ctx, ctx->plan, 2 * (o + bytes)));
    }
    *dev = (char *)ctx->plan.p + o;
    ctx->plan_off = o + bytes;
    return HALIGN_OK;
}

// The next timing triple of this call (created on first use).
int tev_next(halign_ctx *ctx, std::array<hipEvent_t, 3> **out) {
    if (ctx->ntev == (int)ctx->tev.size()) {
        std::array<hipEvent_t, 3> t{};
        for (auto &e : t) HCHK(hipEventCreate(&e));
        ctx->tev.push_back(t);
    }
    *out = &ctx->tev[ctx->ntev++];
    return HALIGN_OK;
}

// Forward and walk time (ms) summed over the triples of the last call
// (synchronises on the last one).
int tev_sum(halign_ctx *ctx, float *fwd, float *walk) {
    *fwd = *walk = 0.f;
    if (ctx->ntev == 0) return HALIGN_OK;
    HCHK(hipEventSynchronize(ctx->tev[ctx->ntev - 1][2]));
    for (int q = 0; q < ctx->ntev; ++q) {
        float f = 0.f, w = 0.f;
        HCHK(hipEventElapsedTime(&f, ctx->tev[q][0], ctx->tev[q][1]));
        HCHK(hipEventElapsedTime(&w, ctx->tev[q][1], ctx->tev[q][2]));
        *fwd += f;
        *walk += w;
    }
    return HALIGN_OK;
}

// A packed plan: host arrays laid out in one staging buffer and copied with
// one H2D transfer into ctx->plan.
struct PlanBuilder {
    std::vector<std::pair<size_t, size_t>> parts;  // (offset, bytes)
    size_t total = 0;
    size_t add(size_t bytes) {
        size_t o = (total + 255) & ~size_t(255);
        parts.push_back({o, bytes});
        total = o + bytes;
        return o;
    }
};

inline int grid_for(int64_t n, int block, int maxg = 65536) {
    int64_t g = (n + block - 1) / block;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, maxg));
}

int launch_fill(uint32_t *p, uint32_t v, int64_t n, hipStream_t st) {
    if (n <= 0) return HALIGN_OK;
    hipLaunchKernelGGL(hk::fill_u32_kernel, dim3(grid_for(n, 256, 4096)), dim3(256), 0, st, p, v, n);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

int check_scoring(const halign_scoring *sc) {
    if (!sc || !sc->matrix_host) return fail(HALIGN_E_INVALID, "scoring is NULL");
    if (sc->alphabet <= 0 || sc->alphabet > hk::kAlphaMax)
        return fail(HALIGN_E_UNSUPPORTED, "alphabet %d outside 1..32", sc->alphabet);
    if (sc->gap_open < 0 || sc->gap_extend < 1)
        return fail(HALIGN_E_UNSUPPORTED, "need gap_open >= 0 and gap_extend >= 1");
    if (sc->gap_open + sc->gap_extend > 1000000)
        return fail(HALIGN_E_UNSUPPORTED, "gap costs too large");
    return HALIGN_OK;
}

// *longest (optional): the longest sequence.
int check_seqs(const halign_seqs *sq, int *longest = nullptr) {
    if (longest) *longest = 0;
    if (!sq || sq->n < 0) return fail(HALIGN_E_INVALID, "seqs is NULL or n < 0");
    if (sq->n == 0) return HALIGN_OK;
    if (!sq->residues || !sq->offsets || !sq->offsets_host)
        return fail(HALIGN_E_INVALID, "seqs pointers are NULL");
    const int64_t *o = sq->offsets_host;
    if (o[0] != 0) return fail(HALIGN_E_INVALID, "offsets[0] must be 0");
    int64_t top = 0;
    for (int k = 0; k < sq->n; ++k) {
        const int64_t L = o[k + 1] - o[k];
        if (L < 0) return fail(HALIGN_E_INVALID, "offsets decrease at %d", k);
        if (L >= 65536) return fail(HALIGN_E_UNSUPPORTED, "sequence %d has length %lld >= 65536", k, (long long)L);
        top = std::max(top, L);
    }
    if (longest) *longest = (int)top;
    return HALIGN_OK;
}

// Device matrix copy (alpha x alpha int8) kept in the plan buffer head.
struct Scoring {
    const int8_t *dmat;
    const int8_t *hmat;   // host copy (planning decisions)
    int alpha, ge, goe;
};

// ---------------------------------------------------------------------------
// Forward + walk for one set of pairs against one center.
// ---------------------------------------------------------------------------
enum Route { kRouteIntra = 0, kRouteInter = 1 };

// pairs longer than this (sequence residues) run on the wavefront kernel even
// in a batch that runs one pair per lane
constexpr int kLongPair = 1000;

// Rows per lane and passes of the wavefront kernel: passes = ceil(m / 512),
// R = ceil(m / (64 * passes)) <= 8, so a pass holds 64*R >= m/passes rows.
void pick_geom(int m, int *R, int *passes) {
    const int p = std::max(1, (m + 511) / 512);
    *passes = p;
    *R = std::max(1, std::min(8, (m + 64 * p - 1) / (64 * p)));
}

// Boundary-row columns per strip-kernel lane: the longest sequence rounded
// up to whole prefetch blocks.
int64_t strip_cols(int nmax_all) {
    return ((int64_t)std::max(1, nmax_all) + hk::kB - 1) / hk::kB * hk::kB;
}

void launch_inter(const hk::InterArgs &a, bool tb, bool endc, int grid, hipStream_t st,
                  const hk::Timed &t = hk::Timed()) {
    if (tb) hk::launch_timed(t, hk::sw_inter_kernel<true, true>, dim3(grid), dim3(64), 0, st, a);
    else if (endc) hk::launch_timed(t, hk::sw_inter_kernel<false, true>, dim3(grid), dim3(64), 0, st, a);
    else hk::launch_timed(t, hk::sw_inter_kernel<false, false>, dim3(grid), dim3(64), 0, st, a);
}

// Geometry of the wavefront forward for a batch.
struct StreamGeom {
    int R = 8, passes = 1, LS = 64, pk = 0;
};

// Lengths by rank, longest first: all of them, or a sample of n of the np.
struct Lens {
    const int32_t *v;
    int n, np;
    int32_t operator[](int rank) const { return n == np ? v[rank] : v[(int64_t)rank * n / np]; }
};

// Streams of a batch of `np` non-empty pairs (lengths plen, longest first) when
// `cap` streams are resident, and the columns that a wavefront's share of them
// takes: the mean of the average and the longest stream (streams end apart,
// and those that end early leave their issue slots to the others).
double stream_cols(const Lens &plen, int np, int64_t sum_len, int cap) {
    if (cap >= np) return 0.5 * ((double)sum_len / np + plen[0]);
    const double avg = (double)sum_len / cap;
    double top = std::max<double>(plen[0], 1.05 * avg);
    if (np < 2 * cap)   // the shortest pairs join the streams of the shortest long ones
        for (int i : {0, (np - cap) / 2, np - cap - 1}) top = std::max<double>(top, plen[cap - 1 - i] + plen[cap + i]);
    return 0.5 * (avg + top);
}

// Cycles that a SIMD needs for the batch with geometry g and `w` wavefronts per
// SIMD of it resident.  A step issues about ops(R) instructions of 4 cycles;
// w wavefronts on a SIMD take kShare[w] issue times per step of each (a serial
// chain alone: 1.28; four together fill the issue slots), and no stream ends
// before its longest pair.  A model for choosing, not for timing: with traceback it gives
// 0.67 to 1.32 of the measured forward time, score-only 0.52 to 1.56 (20,000 pairs of
// 200-500 on m = 311, 4,000 on 450, 300 of 300-900 on 800, 64 of 80-160 on 120,
// 50,001 of a long tail on 101, 300,000 of 50-1000 on 93 and 200, each on the five
// geometries).  The geometry it picks there is the fastest of the five but for the
// long tail with traceback (1.04 ms against 1.00) and 64 scored pairs (45 us against
// 41): packed streams of 32 or 16 lanes where they fill the chip, 64 lanes below.
constexpr double kShare[7] = {1.28, 1.28, 2.2, 3.15, 4, 5, 6};
double stream_cost(const halign_ctx *ctx, const StreamGeom &g, bool tb, const Lens &plen, int np, int64_t sum_len,
                   int w) {
    const int per_wave = 64 / g.LS * (g.pk ? 2 : 1), simds = ctx->num_cu * 4;
    const double ops = g.pk ? (tb ? 17.8 * g.R + 65 : 10.5 * g.R + 65)
                            : (tb ? 16.4 * g.R + 38 : 9.0 * g.R + 30);
    const double cols = stream_cols(plen, np, sum_len, simds * w * per_wave);
    const int waves = (std::min(np, simds * w * per_wave) + per_wave - 1) / per_wave;
    const int weff = (waves + simds - 1) / simds;
    return 4.0 * ops * g.passes *
           std::max((cols + g.LS - 1) * kShare[std::min(6, weff)], (plen[0] + g.LS - 1) * kShare[1]);
}

// Resident wavefronts per SIMD that the packed kernel's streams are sized for
// (stream16_waves fit its registers): that many, or fewer where more pairs per
// stream end closer together by the model, by more than the 3% that runs of such
// numbers differ by (20,000 on m = 311, 32 lanes: 0.77 ms with two and three, 0.79 with four).
// Right to a few per cent on even lengths; on the long tail it takes one wavefront
// where two are faster (1.04 against 0.84 ms).
int packed_waves(const halign_ctx *ctx, const StreamGeom &g, bool tb, const Lens &plen, int np, int64_t sum_len,
                 int wmax) {
    int best = std::min(hk::stream16_waves(g.R, tb), wmax);
    double cost = stream_cost(ctx, g, tb, plen, np, sum_len, best);
    for (int w = best - 1; w >= 1; --w) {
        const double c = stream_cost(ctx, g, tb, plen, np, sum_len, w);
        if (c < 0.97 * cost) {
            cost = c;
            best = w;
        }
    }
    return best;
}

struct BatchOut {
    int32_t *score, *cells, *endcell;
    uint16_t *ins;
    uint32_t *aligned;
    int32_t *G = nullptr;   // optional: max-merge of ins into G during the walk
    int gskip = -1;         // pair left out of G (the center itself)
};

constexpr int kDevPlanMin = 2048;   // pairs from which the device plans a batch
constexpr int kHistParts = 16;      // workgroups that count them
constexpr int kPlanFetch = 1 << 15; // plan bytes up to which a kernel fetches them from the stage

// Plans and runs the forward pass (+ walk when tb) for the pairs `pids_in`
// against center (device) of length m.
struct Tune {
    int route = -1;   // -1: from flags
    int R = 0;        // 0: fitted to m
    int smul = 1;     // streams per resident wave slot
    double scale = 1; // stream count scale (a sample keeps the batch's pairs per stream)
    int LS = 0;       // lanes per stream (0: 64)
    int pk = 0;       // 1: packed 16-bit wavefront kernel (two streams per lane group)
};

// pairs_in: the pair ids of the batch (NULL: 0 .. np-1).
int run_batch(halign_ctx *ctx, const Scoring &S, const uint8_t *center, int m, const halign_seqs *sq,
              const int32_t *pids_in, int np, bool tb, bool endc, int route, const BatchOut &out, hipStream_t st,
              const Tune &tune = Tune(), int dev_longest = -1, bool counted = false) {
    const int64_t *oh = sq->offsets_host;
    if (np == 0) return HALIGN_OK;
    auto pid_of = [&](int x) { return pids_in ? pids_in[x] : x; };
    // Planned on the device (plan_kernels.hpp) from 2,048 pairs, where the caller
    // allows it (dev_longest: the longest of all pairs; counted: the call's first
    // kernel has counted them by length), the batch is not a
    // captured one (whose replays read the host's plan) and the knobs leave the
    // dealing open; the host then only looks at a sample of the lengths.  Below,
    // the host plans faster than the kernels' launches (64 pairs: 5 us).
    bool dev = dev_longest >= 0 && !pids_in && np >= kDevPlanMin && !ctx->capturing && !getenv("HALIGN_DEAL");
    int32_t *pids = nullptr, *plen = nullptr;
    int64_t sum_len = 0;
    int nonempty_all = np;   // (empty pairs sort last)
    // longest first (counting sort on length, stable); plen[x] = length of
    // pids[x], so that later passes read lengths in order
    auto sort_pairs = [&]() {
        if ((int)ctx->h_pids.size() < np) {
            ctx->h_pids.resize(np);
            ctx->h_plen.resize(np);
        }
        pids = ctx->h_pids.data();
        plen = ctx->h_plen.data();
        int maxlen = 0;
        sum_len = 0;
        for (int x = 0; x < np; ++x) {
            const int p = pid_of(x);
            maxlen = std::max(maxlen, (int)(oh[p + 1] - oh[p]));
        }
        std::vector<int32_t> &cnt = ctx->h_cnt;
        cnt.assign(maxlen + 2, 0);
        for (int x = 0; x < np; ++x) {
            const int p = pid_of(x);
            const int L = (int)(oh[p + 1] - oh[p]);
            cnt[maxlen - L]++;
            sum_len += L;
        }
        int acc = 0;
        for (auto &c : cnt) { const int v = c; c = acc; acc += v; }
        for (int x = 0; x < np; ++x) {
            const int p = pid_of(x);
            const int L = (int)(oh[p + 1] - oh[p]);
            const int q = cnt[maxlen - L]++;
            pids[q] = p;
            plen[q] = L;
        }
        nonempty_all = np;
        while (nonempty_all > 0 && plen[nonempty_all - 1] == 0) --nonempty_all;
    };
    Lens lens{nullptr, 0, 0};
    if (dev) {   // a strided sample of 1,024 lengths, sorted, its first one the longest of all
        constexpr int kSample = 1024;
        sum_len = oh[np] - oh[0];
        dev = sum_len > 0;
        std::vector<int32_t> &cnt = ctx->h_cnt, &smp = ctx->h_samp;
        cnt.assign(dev_longest + 1, 0);
        for (int x = 0; x < kSample; ++x) {
            const int p = (int)((int64_t)x * np / kSample);
            cnt[oh[p + 1] - oh[p]]++;
        }
        smp.clear();
        for (int L = dev_longest; L >= 0; --L) smp.insert(smp.end(), cnt[L], L);
        smp[0] = dev_longest;
        lens = Lens{smp.data(), kSample, np};
    }
    if (!dev) {
        sort_pairs();
        lens = Lens{plen, nonempty_all > 0 ? nonempty_all : np, nonempty_all > 0 ? nonempty_all : np};
    }
    hmark(ctx, "sort");
    const int aw = (m + 31) / 32;
    // int16 profile when every score and profile entry fits in 16 bits:
    // max score <= max(S) * min(m, longest sequence)
    int smax = 1;
    for (int x = 0; x < S.alpha * S.alpha; ++x) smax = std::max(smax, (int)S.hmat[x]);
    const int nlong = lens[0];
    const bool p16 = (int64_t)smax * std::min(m, nlong) <= 32000 && S.goe + 128 <= 32000 &&
                     !getenv("HALIGN_PROFILE32");
    int R = 8, passes = 1, LS = 64;
    pick_geom(m, &R, &passes);
    if (tune.route >= 0) route = tune.route;
    // packed 16-bit wavefront kernel: only when every H stays below 15000 and
    // the gap costs are small
    const bool pk_fits = p16 && (int64_t)smax * std::min(m, nlong) < 15000 && S.goe <= 256 && S.ge <= 256;
    bool pk = false;
    auto narrow = [&](int ls) {   // the fewest passes of streams of ls lanes, and the rows that fills
        StreamGeom g;
        g.LS = ls;
        g.passes = std::max(1, (m + ls * 16 - 1) / (ls * 16));
        g.R = std::max(2, (m + ls * g.passes - 1) / (ls * g.passes));
        return g;
    };
    const char *env_ls = getenv("HALIGN_STREAM_LANES");   // test knobs: narrower streams,
    const char *env_pk = getenv("HALIGN_STREAM_PACK");    // and the packed kernel on them
    if (tune.R > 0) {
        if (stream_supported(tune.R, tune.LS > 0 ? tune.LS : 64, p16)) {
            LS = tune.LS > 0 ? tune.LS : 64;
            R = tune.R;
            passes = std::max(1, (m + LS * R - 1) / (LS * R));
        }
        pk = tune.pk > 0 && pk_fits && stream16_supported(R, LS);
    } else if (env_ls) {
        const int ls = atoi(env_ls);
        if ((ls == 32 || ls == 16) && stream_supported(narrow(ls).R, ls, p16)) {
            const StreamGeom g = narrow(ls);
            LS = ls;
            R = g.R;
            passes = g.passes;
        }
        pk = env_pk && atoi(env_pk) != 0 && pk_fits && stream16_supported(R, LS);
    } else if (route == kRouteIntra && p16 && nonempty_all > 0 && !env_pk) {
        // no plan given: the cheapest geometry by stream_cost
        StreamGeom best{R, passes, 64, 0};
        double cost = stream_cost(ctx, best, tb, lens, nonempty_all, sum_len, R > 6 ? 4 : 6);
        for (int ls : {32, 16})
            for (int k = 0; k <= (pk_fits ? 1 : 0); ++k) {
                StreamGeom g = narrow(ls);
                g.pk = k;
                const int w = k ? packed_waves(ctx, g, tb, lens, nonempty_all, sum_len, 4) : (g.R > 6 ? 4 : 6);
                const double c = stream_cost(ctx, g, tb, lens, nonempty_all, sum_len, w);
                if (c < cost) {
                    cost = c;
                    best = g;
                }
            }
        R = best.R;
        passes = best.passes;
        LS = best.LS;
        pk = best.pk != 0;
    }
    pk = pk && route == kRouteIntra;
    const int W = (R + 7) / 8, NS = 64 / LS;
    const int WQ = pk ? (R + 3) / 4 : W;   // code words per step
    const size_t prof_bytes = (size_t)(S.alpha + 1) * LS * (p16 ? 16 * W : 4 * R);
    // wavefronts per workgroup: one per SIMD, so that any number per SIMD spreads
    // evenly over the CUs (300 pairs of 300-900 on m = 800: 0.71 against 1.08 ms);
    // eight in large batches of the 32-bit kernel, which share a profile
    const int wg_waves = pk || (int64_t)nonempty_all <= (int64_t)ctx->num_cu * 16 * NS ? 4 : 8;
    const size_t lds_stream =
        prof_bytes + std::max<size_t>(p16 ? hk::kProfTmp : 0,
                                      tb ? (size_t)wg_waves * 1024 * (pk ? WQ : 2 * W) : (size_t)0);
    const StreamGeom geom{R, passes, LS, pk ? 1 : 0};
    if (route == kRouteIntra && lds_stream > ctx->lds_max) route = kRouteInter;
    ctx->last_stats[2] = route;
    ctx->last_pk = pk ? 1 : 0;
    // streams of a set of pairs (lengths l, longest first): the pairs are dealt
    // over the resident wavefronts so that every stream has about the same
    // columns.  Resident workgroups per CU: by LDS, and by registers (the 32-bit
    // kernel holds four waves per SIMD with R > 6, else six)
    auto count_streams = [&](const Lens &l, int n, int64_t cols) {
        const int wg_lds = std::max(1, (int)((pk ? ctx->lds_cu : ctx->lds_max) / lds_stream));
        const int wg_per_cu = pk ? (n > 0 ? packed_waves(ctx, geom, tb, l, n, cols, wg_lds) : 1)
                                 : std::max(1, std::min({4, wg_lds, (R > 6 ? 4 : 6) * 4 / 8}));
        const int resident = ctx->num_cu * wg_per_cu * (pk ? 4 : 8) * NS * std::max(1, tune.smul) * (pk ? 2 : 1);
        int ns = std::max(1, std::min(n, (int)std::max(1.0, resident * tune.scale)));
        if (const char *e = getenv("HALIGN_MAX_STREAMS")) {   // test knob: many pairs per stream
            const int cap_s = atoi(e);
            if (cap_s > 0) ns = std::min(ns, cap_s);
        }
        return ns;
    };
    // The device's dealing by formula (the dev_own longest pairs on streams of
    // their own, the rest dealt in alternating order) serves where its longest
    // stream, estimated from the sample, is within 30% of the longest pair or of
    // the average stream, and its equal regions take at most four times the
    // columns.  Forward time against dealing to the least loaded stream: batch of
    // 20,000 0.77 ms against 0.79; 300,000 10.7 against 11.1; a long tail of 50,001
    // 0.99-1.04 against 0.885, for 0.23 ms less on the host (whole call 1.25-1.28
    // against 1.34; 1.36 forward without streams of their own).  Up to 64 pairs a
    // stream, whose lengths the staging kernel's wavefronts add with one load a
    // lane.  The host is no faster beyond (1,200,000 pairs in 37 rounds 4.1 ms a call on
    // the device, 13.9 on the host; 2,500,000 in 77 8.4 and 31.8).
    int dev_ns = 0, dev_own = 0;
    int64_t dev_cols = 0;
    size_t dev_code_words = 0, dev_bound = 0;
    const int per_group = pk ? 2 : 1;
    if (dev && route == kRouteIntra) {
        dev_ns = count_streams(lens, np, sum_len);
        const int64_t avg = sum_len / dev_ns;
        const int rounds = (np + dev_ns - 1) / dev_ns;
        dev = rounds <= 64;
        dev_cols = nlong;
        double top = nlong;
        if (dev && rounds > 1) {
            for (int sh : {0, 5, 4, 3}) {   // no pair on its own, or 1/32, 1/16, 1/8 of the streams
                const int k = sh ? dev_ns >> sh : 0, n2 = dev_ns - k;
                double most = nlong;
                for (int q = 0; q <= 4; ++q) {
                    const int s2 = (int)((int64_t)(n2 - 1) * q / 4);
                    double load = 0;
                    for (int64_t r = 0; k + r * n2 < np; ++r) {
                        const int64_t x = k + r * n2 + ((r & 1) ? n2 - 1 - s2 : s2);
                        if (x < np) load += lens[(int)x];
                    }
                    most = std::max(most, load);
                }
                if (sh == 0 || most < 0.95 * top) {
                    top = most;
                    dev_own = k;
                }
            }
            dev_cols = sum_len / (dev_ns - dev_own) + nlong;
        }
        if (tb) dev_code_words = (size_t)passes * (size_t)((dev_cols + LS - 1 + 7) / 8) * LS * 8 * WQ;
        dev_bound = (size_t)(passes - 1) * (size_t)dev_cols;
        const size_t groups = (size_t)(dev_ns + per_group - 1) / per_group;
        dev = dev && top <= 1.3 * (double)std::max<int64_t>(nlong, avg) && dev_cols <= 4 * avg && dev_cols < (1 << 30) &&
              groups * (dev_code_words * 4 + dev_bound * 8) <= (ctx->cap ? ctx->cap : (size_t)1 << 62);
    } else {
        dev = false;
    }
    if (!dev && !pids) {
        sort_pairs();
        lens = Lens{plen, nonempty_all > 0 ? nonempty_all : np, nonempty_all > 0 ? nonempty_all : np};
    }

    const char *deal_env = getenv("HALIGN_DEAL");   // test knob: snake dealing
    const bool deal_lpt = !(deal_env && !strcmp(deal_env, "snake"));
    // chunk the pairs so that codes + boundary rows fit the cap
    const size_t cap = ctx->cap ? ctx->cap : (size_t)1 << 62;
    std::vector<std::pair<int, int>> chunks;  // [lo, hi) in pids
    // columns that the codes cover: every pair's, and a fill and drain per
    // stream (at most one per pair).  Two streams of the packed kernel share
    // theirs, sized by the longer one: dealt to the least loaded, they end
    // within one pair of each other.
    size_t code_cols = (size_t)sum_len + (size_t)(LS + 8) * (size_t)np;
    if (pk && deal_lpt)
        code_cols = std::min(code_cols, ((size_t)sum_len + (size_t)nlong * nonempty_all / 2) / 2 + (size_t)(LS + 8) * np);
    const size_t intra_bytes =
        (tb ? (size_t)passes * LS * 4 * WQ * code_cols : 0) + (size_t)(passes - 1) * 8 * (size_t)sum_len;
    if (dev || (route == kRouteIntra && intra_bytes <= cap)) {
        chunks.push_back({0, np});
    } else {
        const int nst = (m + hk::kT - 1) / hk::kT;
        int lo = 0;
        size_t acc = 0;
        for (int x = 0; x < np; ++x) {
            const int n = plen[x];
            size_t b = 0;
            bool boundary = true;
            if (route == kRouteIntra) {
                b = (tb ? (size_t)passes * (n + LS + 8) * LS * 4 * WQ : 0) + (size_t)(passes - 1) * n * 8;
            } else {
                boundary = (x - lo) % 64 == 0;
                b = (boundary && tb) ? (size_t)nst * ((n + 3) / 4) * 512 * 4 : 0;  // group charged by its longest
            }
            if (boundary && x > lo && acc + b > cap) {
                chunks.push_back({lo, x});
                lo = x;
                acc = 0;
            }
            acc += b;
        }
        chunks.push_back({lo, np});
    }
    ctx->last_stats[3] += (int64_t)chunks.size();
    const int64_t cells_total = (int64_t)m * sum_len;
    ctx->last_stats[0] += cells_total;
    RCHK(grow(ctx, ctx->counter, 256));
    unsigned long long *counter = (unsigned long long *)ctx->counter.p;

    int64_t launches = 0;
    for (size_t ci = 0; ci < chunks.size(); ++ci) {
        const int lo = chunks[ci].first, hi = chunks[ci].second;
        const int cn = hi - lo;
        size_t code_words = 0, bound_elems = 0;   // of the chunk
        int nstreams = 0, nslots = 0, ngroups = 0;
        int64_t total_cols = 0;
        const bool strip_plan = route != kRouteIntra;
        const int chunk_nmax = dev ? nlong : plen[lo];
        // the plan's arrays, as offsets into the chunk's region of the device plan
        size_t o_cbase = 0, o_cstr = 0, o_ccol = 0, o_walk = 0, o_sbeg = 0, o_slen = 0, o_slot0 = 0, o_scb = 0,
               o_sbb = 0, o_spid = 0, o_scol = 0, o_sstr = 0, o_order = 0, o_gnmax = 0, o_gcb = 0;
        char *dplan = nullptr, *zplan = nullptr;
        size_t plan_bytes = 0;
        if (dev) {
            PlanBuilder pb;
            nstreams = dev_ns;
            nslots = cn;
            o_sbeg = pb.add(sizeof(int64_t) * nstreams);
            o_slen = pb.add(sizeof(int32_t) * nstreams);
            o_slot0 = pb.add(sizeof(int32_t) * nstreams);
            o_scb = pb.add(sizeof(int64_t) * nstreams);
            o_sbb = pb.add(sizeof(int64_t) * nstreams);
            o_spid = pb.add(sizeof(int32_t) * nslots);
            o_scol = pb.add(sizeof(int64_t) * nslots);
            o_sstr = pb.add(sizeof(int32_t) * nslots);
            o_order = pb.add(sizeof(int2) * nslots);
            const size_t o_hist = pb.add(sizeof(int32_t) * (nlong + 1));
            RCHK(plan_dev(ctx, pb.total, st, &dplan));
            total_cols = (int64_t)nstreams * dev_cols;
            const size_t groups = (size_t)(nstreams + per_group - 1) / per_group;
            code_words = groups * dev_code_words;
            bound_elems = groups * dev_bound;
            const size_t keys_b = ((size_t)nslots * 8 + 255) & ~size_t(255);
            RCHK(grow(ctx, ctx->sbuf, keys_b + (size_t)total_cols + 64));
            hk::DevPlanArgs d{};
            d.res = sq->residues;
            d.off = sq->offsets;
            d.np = cn;
            d.maxlen = nlong;
            d.ns = nstreams;
            d.own = dev_own;
            d.clamp = S.alpha;
            d.hist = (int32_t *)(dplan + o_hist);
            d.order = (int2 *)(dplan + o_order);
            d.per_group = per_group;
            d.cols = dev_cols;
            d.code_words = (int64_t)dev_code_words;
            d.bound_elems = (int64_t)dev_bound;
            d.spid = (int32_t *)(dplan + o_spid);
            d.sstr = (int32_t *)(dplan + o_sstr);
            d.slot0 = (int32_t *)(dplan + o_slot0);
            d.slen = (int32_t *)(dplan + o_slen);
            d.scol = (int64_t *)(dplan + o_scol);
            d.sbeg = (int64_t *)(dplan + o_sbeg);
            d.scb = (int64_t *)(dplan + o_scb);
            d.sbb = (int64_t *)(dplan + o_sbb);
            d.keys = (unsigned long long *)ctx->sbuf.p;
            d.sres = (uint8_t *)ctx->sbuf.p + keys_b;
            if (!counted) {
                RCHK(launch_fill((uint32_t *)d.hist, 0u, nlong + 1, st));
                hipLaunchKernelGGL(hk::plan_hist_kernel, dim3(grid_for(cn, 1024, 128)), dim3(256), 0, st, d);
            }
            hipLaunchKernelGGL(hk::plan_scan_kernel, dim3(1), dim3(1024), 0, st, d.hist, nlong,
                               counted ? (const int32_t *)ctx->histbuf.p : nullptr, counted ? kHistParts : 0);
            hipLaunchKernelGGL(hk::plan_scatter_kernel, dim3(grid_for(cn, 1024 * hk::kScatterPer, 1 << 30)), dim3(1024), 0,
                               st, d);
            hipLaunchKernelGGL(hk::plan_stage_kernel, dim3((unsigned)((cn + 3) / 4)), dim3(256), 0, st, d);
            HCHK(hipGetLastError());
            hmark(ctx, dev_own > 0 ? "dplan_own" : "dplan");
        } else {
            PlanBuilder pb;
            // strip route: the walk list and its walk descriptors, both in walk
            // order (the wavefront route's walk reads the per-slot and per-stream
            // plan)
            o_cbase = strip_plan ? pb.add(sizeof(int64_t) * cn) : 0;
            o_cstr = strip_plan ? pb.add(sizeof(int32_t) * cn) : 0;
            o_ccol = strip_plan ? pb.add(sizeof(int32_t) * cn) : 0;
            o_walk = strip_plan ? pb.add(sizeof(int32_t) * cn) : 0;
            int64_t ch_len = 0;
            int nonempty = 0;   // pairs [0, nonempty) of the chunk are non-empty: empty pairs sort last
            for (int x = hi - 1; x >= lo && plen[x] == 0; --x) ++nonempty;
            nonempty = cn - nonempty;
            if (route == kRouteIntra) {
                for (int x = 0; x < nonempty; ++x) ch_len += plen[lo + x];
                nstreams = count_streams(Lens{plen + lo, nonempty, nonempty}, nonempty, ch_len);
                nslots = cn;
                o_sbeg = pb.add(sizeof(int64_t) * nstreams);
                o_slen = pb.add(sizeof(int32_t) * nstreams);
                o_slot0 = pb.add(sizeof(int32_t) * nstreams);
                o_scb = pb.add(sizeof(int64_t) * nstreams);
                o_sbb = pb.add(sizeof(int64_t) * nstreams);
                o_spid = pb.add(sizeof(int32_t) * nslots);
                o_scol = pb.add(sizeof(int64_t) * nslots);
                o_sstr = pb.add(sizeof(int32_t) * nslots);
            } else {
                ngroups = (cn + 63) / 64;
                o_order = pb.add(sizeof(int32_t) * (size_t)ngroups * 64);
                o_gnmax = pb.add(sizeof(int32_t) * ngroups);
                o_gcb = pb.add(sizeof(int64_t) * ngroups);
            }
            char *hs = nullptr;
            pb.total = (pb.total + 15) & ~size_t(15);
            RCHK(stage_host(ctx, pb.total, &hs));
            int32_t *h_walk = (int32_t *)(hs + o_walk);
            int64_t *h_cbase = (int64_t *)(hs + o_cbase);
            int32_t *h_cstr = (int32_t *)(hs + o_cstr);
            int32_t *h_ccol = (int32_t *)(hs + o_ccol);
            if (strip_plan)
                for (int x = 0; x < cn; ++x) h_walk[x] = pids[lo + x];
            if (route == kRouteIntra) {
                int64_t *h_sbeg = (int64_t *)(hs + o_sbeg);
                int32_t *h_slot0 = (int32_t *)(hs + o_slot0);
                int64_t *h_scb = (int64_t *)(hs + o_scb);
                int64_t *h_sbb = (int64_t *)(hs + o_sbb);
                int32_t *h_spid = (int32_t *)(hs + o_spid);
                int64_t *h_scol = (int64_t *)(hs + o_scol);
                int32_t *h_sstr = (int32_t *)(hs + o_sstr);   // stream of each slot (for the walk)
                // pairs and columns of each stream, then slots grouped by stream.
                // Snake dealing: the k-th non-empty pair, k = r * nstreams + q, goes
                // to stream q in even rounds r and nstreams - 1 - q in odd ones.
                // Least-loaded dealing: each pair (longest first) goes to the stream
                // with the fewest columns so far (a bucket queue on the column
                // count, whose minimum only grows), so streams end within one pair
                // length of each other.
                std::vector<int32_t> &scount = ctx->h_scount;
                std::vector<int64_t> &scols = ctx->h_scols;
                scount.assign(nstreams, 0);
                scols.assign(nstreams, 0);
                std::vector<int32_t> &sof = ctx->h_sof;   // least-loaded dealing: stream of each non-empty pair
                const int64_t maxload = (nonempty > 0 ? ch_len / nstreams + plen[lo] : 0) + 1;
                const bool lpt = deal_lpt && maxload <= ((int64_t)1 << 22);
                hmark(ctx, "p_setup");
                if (lpt) {
                    if ((int)sof.size() < nonempty) sof.resize(nonempty);
                    std::vector<int32_t> &head = ctx->h_head, &nxt = ctx->h_nxt;
                    head.assign(maxload + 1, -1);
                    if ((int)nxt.size() < nstreams) nxt.resize(nstreams);
                    for (int s2 = 0; s2 < nstreams; ++s2) nxt[s2] = s2 + 1 < nstreams ? s2 + 1 : -1;
                    head[0] = 0;
                    int64_t minp = 0;
                    for (int x = 0; x < nonempty; ++x) {
                        while (head[minp] < 0) ++minp;
                        const int s2 = head[minp];
                        head[minp] = nxt[s2];
                        sof[x] = s2;
                        scount[s2]++;
                        scols[s2] += plen[lo + x];
                        const int64_t l2 = minp + plen[lo + x];
                        nxt[s2] = head[l2];
                        head[l2] = s2;
                    }
                } else {
                    int r = 0, q = 0;   // round and position of the next non-empty pair
                    for (int x = 0; x < nonempty; ++x) {
                        const int s2 = (r & 1) ? nstreams - 1 - q : q;
                        scount[s2]++;
                        scols[s2] += plen[lo + x];
                        if (++q == nstreams) { q = 0; ++r; }
                    }
                }
                hmark(ctx, "p_deal");
                int slot = 0;
                int64_t col = 0;
                for (int s = 0; s < nstreams; ++s) {
                    h_slot0[s] = slot;
                    h_sbeg[s] = col;
                    ((int32_t *)(hs + o_slen))[s] = (int32_t)scols[s];
                    slot += scount[s];
                    col += scols[s];
                    h_scb[s] = (int64_t)code_words;
                    h_sbb[s] = (int64_t)bound_elems;
                    if (pk) {
                        // stream pair (s, s+1) shares the tiles and boundary rows of a
                        // lane group, sized by the longer stream
                        if (s & 1) {
                            h_scb[s] = h_scb[s - 1];
                            h_sbb[s] = h_sbb[s - 1];
                            continue;
                        }
                        const int64_t cq = std::max(scols[s], s + 1 < nstreams ? scols[s + 1] : (int64_t)0);
                        if (tb) code_words += (size_t)passes * ((cq + LS - 1 + 7) / 8) * LS * 8 * WQ;
                        if (passes > 1) bound_elems += (size_t)(passes - 1) * cq;
                        continue;
                    }
                    if (tb) code_words += (size_t)passes * ((scols[s] + LS - 1 + 7) / 8) * LS * 8 * W;
                    if (passes > 1) bound_elems += (size_t)(passes - 1) * scols[s];
                }
                total_cols = col;
                hmark(ctx, "p_streams");
                if (lpt) {
                    // slots of each stream in dealing order (longest first): the
                    // pairs are sorted by stream in host memory first, so that the
                    // pinned plan is written sequentially
                    std::vector<int32_t> &cur = ctx->h_cur, &ord = ctx->h_nxt;
                    cur.assign(h_slot0, h_slot0 + nstreams);
                    if ((int)ord.size() < nonempty) ord.resize(nonempty);
                    for (int x = 0; x < nonempty; ++x) ord[cur[sof[x]]++] = x;
                    for (int s2 = 0, qs = 0; s2 < nstreams; ++s2) {
                        int64_t c = h_sbeg[s2];
                        for (int pl = 0; pl < scount[s2]; ++pl, ++qs) {
                            const int x = ord[qs];
                            h_spid[qs] = pids[lo + x];
                            h_scol[qs] = c;
                            h_sstr[qs] = s2;
                            c += plen[lo + x];
                        }
                    }
                } else {
                    // slots stream by stream (sequential writes): the pl-th pair of
                    // stream s is non-empty pair pl * nstreams + (pl odd ? nstreams - 1 - s : s)
                    for (int s = 0; s < nstreams; ++s) {
                        int64_t c = h_sbeg[s];
                        for (int pl = 0, qs = h_slot0[s]; pl < scount[s]; ++pl, ++qs) {
                            const int x = pl * nstreams + ((pl & 1) ? nstreams - 1 - s : s);
                            h_spid[qs] = pids[lo + x];
                            h_scol[qs] = c;
                            h_sstr[qs] = s;
                            c += plen[lo + x];
                        }
                    }
                }
                for (int x = nonempty; x < cn; ++x) {   // empty pairs after the streamed ones
                    h_spid[x] = pids[lo + x];
                    h_scol[x] = 0;
                    h_sstr[x] = 0;
                }
            } else {
                int32_t *h_order = (int32_t *)(hs + o_order);
                int32_t *h_gnmax = (int32_t *)(hs + o_gnmax);
                int64_t *h_gcb = (int64_t *)(hs + o_gcb);
                const int nst = (m + hk::kT - 1) / hk::kT;
                for (int g = 0; g < ngroups; ++g) {
                    int nmax = 0;
                    for (int l = 0; l < 64; ++l) {
                        const int x = lo + g * 64 + l;
                        h_order[g * 64 + l] = x < hi ? pids[x] : -1;
                        if (x < hi) nmax = std::max(nmax, plen[x]);
                    }
                    h_gnmax[g] = nmax;
                    h_gcb[g] = (int64_t)code_words;
                    // walk entry q = g * 64 + l is the pair in lane l of group g
                    for (int l = 0; l < 64 && lo + g * 64 + l < hi; ++l) {
                        const int q = g * 64 + l;
                        h_cbase[q] = (int64_t)code_words;
                        h_ccol[q] = l;
                        h_cstr[q] = nmax;
                    }
                    if (tb) code_words += (size_t)nst * ((nmax + 3) / 4) * 512;
                }
            }
            hmark(ctx, "plan");
            RCHK(plan_dev(ctx, pb.total, st, &dplan));
            // a small plan goes with the residues' staging (stage_stream_kernel)
            if (route == kRouteIntra && pb.total <= (size_t)kPlanFetch && !ctx->capturing) zplan = (char *)stage_dev(ctx, hs);
            plan_bytes = pb.total;
            if (!zplan) HCHK(hipMemcpyAsync(dplan, hs, pb.total, hipMemcpyHostToDevice, st));
            stage_copied(ctx);
        }
        std::array<hipEvent_t, 3> *tv = nullptr;
        RCHK(tev_next(ctx, &tv));
        hk::Timed tfwd, tend;   // (none while a graph is captured)
        if (!ctx->capturing) {
            tfwd = hk::Timed{(*tv)[0], (*tv)[1]};
            tend = hk::Timed{nullptr, (*tv)[2]};
        }

        if (tb) RCHK(grow(ctx, ctx->codes, std::max<size_t>(4, code_words * 4)));
        if (ctx->fault_chunk == (int)ci) {
            ctx->fault_chunk = -1;
            return fail(HALIGN_E_DEVICE, "injected failure in chunk %d", (int)ci);
        }
        if (route == kRouteIntra) {
            // staged stream residues and per-slot keys share one scratch buffer
            const size_t keys_b = ((size_t)nslots * 8 + 255) & ~size_t(255);
            RCHK(grow(ctx, ctx->sbuf, keys_b + (size_t)total_cols + 64));
            unsigned long long *keys = (unsigned long long *)ctx->sbuf.p;
            uint8_t *sres = (uint8_t *)ctx->sbuf.p + keys_b;
            if (passes > 1) RCHK(grow(ctx, ctx->bound, std::max<size_t>(8, bound_elems * 8)));
            if (!dev) {
                const char *pl = zplan ? zplan : dplan;
                const int n16 = zplan ? (int)(plan_bytes / 16) : 0;
                hipLaunchKernelGGL(hk::stage_stream_kernel, dim3((nslots + 3) / 4 + (n16 + 255) / 256), dim3(256), 0, st,
                                   sq->residues, sq->offsets, (const int32_t *)(pl + o_spid),
                                   (const int64_t *)(pl + o_scol), nslots, S.alpha, sres, keys,
                                   (const uint4 *)zplan, (uint4 *)dplan, n16);
                HCHK(hipGetLastError());
            }
            hk::StreamArgs a{};
            a.mat = S.dmat;
            a.alpha = S.alpha;
            a.center = center;
            a.m = m;
            a.passes = passes;
            a.sres = sres;
            a.sbeg = (const int64_t *)(dplan + o_sbeg);
            a.slen = (const int32_t *)(dplan + o_slen);
            a.nstreams = nstreams;
            a.ge = S.ge;
            a.goe = S.goe;
            a.keys = keys;
            a.sslot0 = (const int32_t *)(dplan + o_slot0);
            a.codes = tb ? (uint32_t *)ctx->codes.p : nullptr;
            a.scbase = (const int64_t *)(dplan + o_scb);
            a.bound = (int2 *)ctx->bound.p;
            a.sbbase = (const int64_t *)(dplan + o_sbb);
            const int waves = ((pk ? (nstreams + 1) / 2 : nstreams) + NS - 1) / NS;
            const int grid = (waves + wg_waves - 1) / wg_waves;
            if (pk) launch_stream16(R, LS, a, tb, grid, wg_waves * 64, lds_stream, st, tfwd);
            else launch_stream(R, LS, a, tb, endc, p16, grid, wg_waves * 64, lds_stream, st, tfwd);
            HCHK(hipGetLastError());
            if (!tb) {   // (with traceback the walk reads the keys)
                hk::launch_timed(tend, hk::decode_keys_kernel, dim3(grid_for(nslots, 256, 1 << 30)), dim3(256), 0, st,
                                 (const unsigned long long *)keys, (const int32_t *)(dplan + o_spid), nslots, out.score,
                                 endc ? out.endcell : (int32_t *)nullptr, (int4 *)out.cells);
                HCHK(hipGetLastError());
            }
        } else {
            const int slots = ctx->num_cu * 16;
            const int grid = std::max(1, std::min(ngroups, slots));
            RCHK(grow(ctx, ctx->bound, (size_t)grid * 64 * strip_cols(chunk_nmax) * 8));
            RCHK(launch_fill((uint32_t *)counter, 0u, 2, st));
            hk::InterArgs a{};
            a.mat = S.dmat;
            a.alpha = S.alpha;
            a.center = center;
            a.m = m;
            a.res = sq->residues;
            a.off = sq->offsets;
            a.mode = 0;
            a.order = (const int32_t *)(dplan + o_order);
            a.gnmax = (const int32_t *)(dplan + o_gnmax);
            a.ngroups = ngroups;
            a.ge = S.ge;
            a.goe = S.goe;
            a.counter = counter;
            a.score = out.score;
            a.endcell = out.endcell;
            a.codes = tb ? (uint32_t *)ctx->codes.p : nullptr;
            a.gcode_base = (const int64_t *)(dplan + o_gcb);
            a.bound = (int2 *)ctx->bound.p;
            a.bstride = (int64_t)64 * strip_cols(chunk_nmax);
            launch_inter(a, tb, endc, grid, st, tfwd);
            HCHK(hipGetLastError());
        }
        ++launches;
        if (tb) {
            hk::WalkArgs w{};
            w.mat = S.dmat;
            w.alpha = S.alpha;
            w.center = center;
            w.m = m;
            w.res = sq->residues;
            w.off = sq->offsets;
            w.pids = strip_plan ? (const int32_t *)(dplan + o_walk) : nullptr;
            w.npairs = cn;
            if (!strip_plan) {
                w.slot_pid = (const int32_t *)(dplan + o_spid);
                w.slot_col = (const int64_t *)(dplan + o_scol);
                w.sbeg = (const int64_t *)(dplan + o_sbeg);
                w.slen = (const int32_t *)(dplan + o_slen);
                w.keys = (const unsigned long long *)ctx->sbuf.p;
                w.slot0 = (const int32_t *)(dplan + o_slot0);
                w.slot_stream = (const int32_t *)(dplan + o_sstr);
                w.scb = (const int64_t *)(dplan + o_scb);
                w.nstreams = nstreams;
            }
            w.ge = S.ge;
            w.goe = S.goe;
            w.score = out.score;
            w.endcell = out.endcell;
            w.codes = (const uint32_t *)ctx->codes.p;
            w.cbase = strip_plan ? (const int64_t *)(dplan + o_cbase) : nullptr;
            w.cstride = strip_plan ? (const int32_t *)(dplan + o_cstr) : nullptr;
            w.ccol = strip_plan ? (const int32_t *)(dplan + o_ccol) : nullptr;
            w.R = R;
            w.lg_ls = LS == 64 ? 6 : (LS == 32 ? 5 : 4);
            w.W = WQ;
            w.kind = route == kRouteIntra ? 0 : 1;
            w.cells = out.cells;
            w.ins = out.ins;
            w.aligned = out.aligned;
            w.aw = aw;
            w.G = out.G;
            w.gskip = out.gskip;
            // cached chunk shape: about as many rows (NB blocks of R rows) as
            // columns (NG chunk columns of 8 or 4), NB * NG = 16
            const int wR = route == kRouteIntra ? R : 16;
            w.rmagic = wR >= 2 ? (uint32_t)((((uint64_t)1 << 32) + wR - 1) / wR) : 0u;
            w.lg_nb = route == kRouteIntra ? (wR >= 4 ? 2 : (wR >= 2 ? 3 : 4)) : 1;
            const dim3 wg(grid_for(cn, hk::kWalkPairs, 1 << 30));
            const bool cl = m <= hk::kWalkCenterLds;
            w.glds = (out.G && m < hk::kWalkGLds) ? 1 : 0;
            const size_t wlds = hk::walk_lds_bytes(route == kRouteIntra ? WQ : 1, m, cl, w.glds != 0);
            if (route == kRouteIntra) {
                if (pk) {
                    if (cl) hk::launch_timed(tend, (hk::walk_kernel<false, true, true>), wg, dim3(256), wlds, st, w);
                    else hk::launch_timed(tend, (hk::walk_kernel<false, false, true>), wg, dim3(256), wlds, st, w);
                } else {
                    if (cl) hk::launch_timed(tend, (hk::walk_kernel<false, true, false>), wg, dim3(256), wlds, st, w);
                    else hk::launch_timed(tend, (hk::walk_kernel<false, false, false>), wg, dim3(256), wlds, st, w);
                }
            } else {
                if (cl) hk::launch_timed(tend, (hk::walk_kernel<true, true, false>), wg, dim3(256), wlds, st, w);
                else hk::launch_timed(tend, (hk::walk_kernel<true, false, false>), wg, dim3(256), wlds, st, w);
            }
            HCHK(hipGetLastError());
        } else if (route != kRouteIntra) {
            RCHK(record(ctx, (*tv)[2], st));
        }
        hmark(ctx, "launch");
        if (ctx->progress && chunks.size() > 1 && !ctx->capturing) {
            // progress lines wait for each chunk; otherwise the host plans the
            // next chunk while this one runs
            HCHK(hipEventSynchronize((*tv)[2]));
            float f = 0, w2 = 0;
            HCHK(hipEventElapsedTime(&f, (*tv)[0], (*tv)[1]));
            HCHK(hipEventElapsedTime(&w2, (*tv)[1], (*tv)[2]));
            fprintf(stderr, "halign: chunk %d/%d done (%d pairs, forward %.1f ms, walk %.1f ms)\n", (int)ci + 1,
                    (int)chunks.size(), cn, f, w2);
            fflush(stderr);
        }
    }
    ctx->last_stats[1] += launches;
    return HALIGN_OK;
}

// ---------------------------------------------------------------------------
// Autotuner: for a bucket of (center length, batch size, median sequence
// length, traceback) it times the candidate plans on a strided sample of the
// batch (every plan gives bit-identical results) and keeps the fastest.
// ---------------------------------------------------------------------------
std::string tune_key(int m, int N, int mean_len, bool tb) {
    int lg = 0;
    while ((1 << (lg + 1)) <= N) ++lg;
    std::ostringstream o;
    o << "m" << (m + 31) / 32 << "_n" << lg << "_l" << (mean_len + 63) / 64 << "_t" << (tb ? 1 : 0);
    return o.str();
}

void tune_load(halign_ctx *ctx) {
    if (ctx->tune_file.empty()) return;
    std::ifstream f(ctx->tune_file);
    std::string line;
    while (std::getline(f, line)) {
        std::istringstream s(line);
        std::string key;
        int r = -1, R = -1, sm = -1, ls = 64, pk = 0;
        if (!(s >> key >> r >> R >> sm)) continue;              // malformed: ignored
        if (!(s >> ls)) ls = 64;                                // lines without the lane count
        if (!(s >> pk)) pk = 0;                                 // lines without the packed flag
        if (r < 0 || r > 1 || R < 0 || R > 16 || sm < 1 || sm > 4 || (ls != 64 && ls != 32 && ls != 16) || pk < 0 ||
            pk > 1)
            continue;
        ctx->tuned[key] = {r, R, sm, ls, pk};
    }
}

void tune_save(halign_ctx *ctx, const std::string &key, const std::array<int, 5> &v) {
    if (ctx->tune_file.empty()) return;
    std::ofstream f(ctx->tune_file, std::ios::app);
    if (f) f << key << " " << v[0] << " " << v[1] << " " << v[2] << " " << v[3] << " " << v[4] << "\n";
}

// *ran: whether candidate plans were run (the stage is then drained).
// dev_longest: as in run_batch; the whole batch is timed under the planner that will run it
// (a sample's ids are planned on the host).
int autotune(halign_ctx *ctx, const Scoring &S, const uint8_t *center, int m, const halign_seqs *sq, bool tb,
             bool endc, const BatchOut &out, int dev_longest, hipStream_t st, Tune *best, bool *ran) {
    *ran = false;
    const int N = sq->n;
    const int mean = N > 0 ? (int)((sq->offsets_host[N] - sq->offsets_host[0]) / N) : 0;
    auto apply = [&](const std::array<int, 5> &v) {
        best->route = v[0];
        best->R = v[1];
        best->smul = v[2];
        best->LS = v[3];
        best->pk = v[4];
    };
    const int64_t ik[4] = {m, N, mean, tb ? 1 : 0};
    if (std::equal(ik, ik + 4, ctx->tkey)) {   // same bucket as the last call: no string key
        apply(ctx->tval);
        return HALIGN_OK;
    }
    const std::string key = tune_key(m, N, mean, tb);
    auto it = ctx->tuned.find(key);
    if (it != ctx->tuned.end()) {
        apply(it->second);
        std::copy(ik, ik + 4, ctx->tkey);
        ctx->tval = it->second;
        return HALIGN_OK;
    }
    *ran = true;
    // the trials write their plans into the stage from its start, where the matrix
    // of this call may still be on its way from
    HCHK(hipStreamSynchronize(st));
    ctx->stage_pending = false;
    // the batch itself (up to 4e10 cells: a few tens of ms per candidate), or a
    // strided sample of 65,536 pairs that keeps the length mix and, through the
    // stream count, the number of pairs per stream
    const double bcells = (double)m * (double)(sq->offsets_host[N] - sq->offsets_host[0]);
    const int ns = bcells <= 4e10 ? N : std::min(N, 65536);
    std::vector<int32_t> sample(ns < N ? ns : 0);
    for (size_t q = 0; q < sample.size(); ++q) sample[q] = (int32_t)((int64_t)q * N / ns);
    int R0 = 8, p0 = 1;
    pick_geom(m, &R0, &p0);
    const double scale = (double)ns / N;
    std::vector<Tune> cands;
    cands.push_back({kRouteIntra, R0, 1, scale, 64});
    cands.push_back({kRouteIntra, R0, 2, scale, 64});
    if (R0 < 8) cands.push_back({kRouteIntra, R0 + 1, 1, scale, 64});
    // narrower streams: fewer fill/drain steps, more rows per lane (int16 profile only;
    // run_batch falls back to 64 lanes otherwise)
    for (int ls : {32, 16}) {
        const int ps = std::max(1, (m + ls * 16 - 1) / (ls * 16));
        const int r = std::max(2, (m + ls * ps - 1) / (ls * ps));
        cands.push_back({kRouteIntra, r, 1, scale, ls});
        // the packed 16-bit kernel on the same geometry (run_batch falls back to
        // the 32-bit one where it does not apply)
        cands.push_back({kRouteIntra, r, 1, scale, ls, 1});
    }
    cands.push_back({kRouteInter, 0, 1, scale, 64});
    // the forward kernels are timed in the same traceback mode as the call
    float best_ms = 1e30f;
    *best = cands[0];
    for (const Tune &c : cands) {
        float ms = 0.f;
        for (int rep = 0; rep < 2; ++rep) {
            // every candidate run starts the stage and the timing triples anew
            // (the previous run has synchronised)
            ctx->stage_off = ctx->plan_off = 0;
            ctx->ntev = 0;
            RCHK(run_batch(ctx, S, center, m, sq, sample.empty() ? nullptr : sample.data(), ns, tb, endc, c.route, out, st,
                           c, dev_longest));
            float wk = 0.f;
            RCHK(tev_sum(ctx, &ms, &wk));
            ctx->stage_pending = false;   // the last event follows the plan's copy
        }
        if (ms < best_ms) {
            best_ms = ms;
            *best = c;
        }
    }
    best->scale = 1;
    const std::array<int, 5> v = {best->route, best->R, best->smul, best->LS > 0 ? best->LS : 64, best->pk};
    ctx->tuned[key] = v;
    tune_save(ctx, key, v);
    std::copy(ik, ik + 4, ctx->tkey);
    ctx->tval = v;
    return HALIGN_OK;
}

// The first staging step of every call: starts the call's stage regions.
// prep (optional): the call's first kernel fetches the matrix itself.
int upload_matrix(halign_ctx *ctx, const halign_scoring *sc, hipStream_t st, Scoring *S,
                  hk::PrepArgs *prep = nullptr) {
    const size_t bytes = (size_t)sc->alphabet * sc->alphabet;
    RCHK(stage_begin(ctx));
    if (ctx->capturing) {   // the device copy from the uncaptured run is kept by the graph
        S->dmat = (const int8_t *)ctx->spbuf.p;
        S->hmat = sc->matrix_host;
        S->alpha = sc->alphabet;
        S->ge = sc->gap_extend;
        S->goe = sc->gap_open + sc->gap_extend;
        return HALIGN_OK;
    }
    RCHK(grow(ctx, ctx->spbuf, 4096));
    char *hs = nullptr;
    RCHK(stage_host(ctx, (bytes + 3) & ~size_t(3), &hs));
    memcpy(hs, sc->matrix_host, bytes);
    if (prep && stage_dev(ctx, hs)) {
        prep->msrc = (const uint32_t *)stage_dev(ctx, hs);
        prep->mdst = (uint32_t *)ctx->spbuf.p;
        prep->mwords = (int)((bytes + 3) / 4);
    } else {
        HCHK(hipMemcpyAsync(ctx->spbuf.p, hs, bytes, hipMemcpyHostToDevice, st));
    }
    stage_copied(ctx);
    S->dmat = (const int8_t *)ctx->spbuf.p;
    S->hmat = sc->matrix_host;
    S->alpha = sc->alphabet;
    S->ge = sc->gap_extend;
    S->goe = sc->gap_open + sc->gap_extend;
    return HALIGN_OK;
}

// Every residue code must be below the alphabet size (HALIGN_E_INVALID).
// The check is enqueued without waiting: the kernels are memory-safe for any
// code (they mask codes to 5 bits), and its result comes to flag_host (by
// flag_fetch, or with the merge's width) for validate_check() to read after the
// call's synchronisation point.  with: what else the launch does.
int validate_codes(halign_ctx *ctx, int alpha, const uint8_t *res, int64_t nres, const uint8_t *center, int m,
                   hipStream_t st, const hk::PrepArgs &with = hk::PrepArgs{}) {
    RCHK(grow(ctx, ctx->counter, 256));
    uint32_t *flag = (uint32_t *)ctx->counter.p + 8;
    // the flag holds (call tag << 8 | largest code) and is raised with
    // atomicMax: a larger tag per call replaces the last call's value without
    // a clearing launch (cleared once when the 24-bit tag wraps).  A captured
    // graph clears the flag itself and uses tag 0 on every replay.
    uint32_t tag = 0;
    if (ctx->capturing) {
        RCHK(launch_fill(flag, 0u, 1, st));
    } else {
        // a buffer not yet cleared here (new, or swapped in) holds stale
        // bytes that would outrank or mimic a tag: clear it first
        if (ctx->vflag != flag || ctx->vtag + 1 >= (1u << 24)) {
            RCHK(launch_fill(flag, 0u, 1, st));
            ctx->vflag = flag;
            ctx->vtag = 0;
        }
        tag = ++ctx->vtag;
    }
    ctx->check_tag = tag;
    hk::PrepArgs a = with;
    a.n = nres > 0 ? nres : 0;
    a.nq = (center && m > 0) ? m : 0;
    a.p = res;
    a.q = center;
    a.tag = tag << 8;
    a.out = flag;
    int64_t work = (a.n + 15) / 16 + 1;
    for (int r = 0; r < 4; ++r) work += a.nz[r] / 4;
    hipLaunchKernelGGL(hk::prep_kernel, dim3(grid_for(work, 256, 1024) + a.hwgs), dim3(256),
                       a.hwgs ? 4 * (size_t)(a.maxlen + 1) : 0, st, a);
    HCHK(hipGetLastError());
    ctx->flag_alpha = alpha;
    return HALIGN_OK;
}

// The check's result to the host: flag_host holds it once the stream has passed.
int flag_fetch(halign_ctx *ctx, hipStream_t st) {
    HCHK(hipMemcpyAsync(ctx->flag_host, (uint32_t *)ctx->counter.p + 8, 4, hipMemcpyDeviceToHost, st));
    return HALIGN_OK;
}

// Call after the stream has synchronised past validate_codes().
int validate_check(halign_ctx *ctx) {
    if (!ctx->flag_alpha) return HALIGN_OK;
    const uint32_t v = (uint32_t)*ctx->flag_host;
    const int h = (v >> 8) == ctx->check_tag ? (int)(v & 0xffu) : 0, alpha = ctx->flag_alpha;
    ctx->flag_alpha = 0;
    if (h >= alpha) return fail(HALIGN_E_INVALID, "residue code %d >= alphabet %d", h, alpha);
    return HALIGN_OK;
}

int validate_now(halign_ctx *ctx, int alpha, const uint8_t *res, int64_t nres, const uint8_t *center, int m,
                 hipStream_t st) {
    RCHK(validate_codes(ctx, alpha, res, nres, center, m, st));
    RCHK(flag_fetch(ctx, st));
    HCHK(hipStreamSynchronize(st));
    ctx->stage_pending = false;   // whatever was copied on the stream has been read
    return validate_check(ctx);
}

// Streams, unless there are pairs enough for every lane of the chip (4 waves
// per SIMD) and their scores need 32 bits (16 with traceback), where one pair
// per lane does as well or better.  300,000 pairs with traceback on a center of
// 200 (93): packed streams 11.4 (5.1) ms, 32-bit streams of 16 lanes 16.7
// (8.5), one pair per lane 20.7 (10.1); 270,000 pairs score-only on 200: packed
// streams 3.7 ms, one pair per lane 7.3.
int route_of(uint32_t flags, const halign_scoring *sc, int m, const halign_seqs *sq, bool tb, int longest) {
    const uint32_t r = flags & (3u << 4);
    if (r == HALIGN_ROUTE_INTER) return kRouteInter;
    if (r == HALIGN_ROUTE_INTRA) return kRouteIntra;
    if (const char *e = getenv("HALIGN_ROUTE")) {
        if (!strcmp(e, "intra")) return kRouteIntra;
        if (!strcmp(e, "inter")) return kRouteInter;
    }
    if (sq->n < 64 * 4 * 1024) return kRouteIntra;
    int smax = 1;
    for (int x = 0; x < sc->alphabet * sc->alphabet; ++x) smax = std::max(smax, (int)sc->matrix_host[x]);
    const int64_t top = (int64_t)smax * std::min(m, longest);
    if (tb) return top <= 32000 ? kRouteIntra : kRouteInter;
    return top < 15000 && sc->gap_open + sc->gap_extend <= 256 ? kRouteIntra : kRouteInter;
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char *halign_last_error(void) { return g_err; }

int halign_ctx_create(int device, size_t workspace_cap_bytes, halign_ctx **out) {
    if (!out) return fail(HALIGN_E_INVALID, "out is NULL");
    *out = nullptr;
    int ndev = 0;
    HCHK(hipGetDeviceCount(&ndev));
    if (device < 0 || device >= ndev) return fail(HALIGN_E_INVALID, "device %d of %d", device, ndev);
    HCHK(hipSetDevice(device));
    halign_ctx *ctx = new (std::nothrow) halign_ctx();
    if (!ctx) return fail(HALIGN_E_NOMEM, "host allocation failed");
    ctx->device = device;
    ctx->cap = workspace_cap_bytes;
    if (ctx->cap == 0) {   // default: a quarter of the memory free at creation
        size_t fr = 0, tot = 0;
        if (hipMemGetInfo(&fr, &tot) == hipSuccess && fr > 0) ctx->cap = fr / 4;
    }
    if (const char *e = getenv("HALIGN_AUTOTUNE")) ctx->autotune = atoi(e) != 0;
    if (const char *e = getenv("HALIGN_PROGRESS")) ctx->progress = atoi(e) != 0;
    if (const char *e = getenv("HALIGN_HOST_TIMING")) ctx->host_timing = atoi(e) != 0;
    if (const char *e = getenv("HALIGN_TUNE_CACHE")) ctx->tune_file = e;
    tune_load(ctx);
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) == hipSuccess) {
        ctx->num_cu = prop.multiProcessorCount;
        ctx->lds_max = prop.maxSharedMemoryPerMultiProcessor ? prop.maxSharedMemoryPerMultiProcessor
                                                             : prop.sharedMemPerBlock;
        if (prop.sharedMemPerBlock && prop.sharedMemPerBlock < ctx->lds_max) ctx->lds_max = prop.sharedMemPerBlock;
        // row emission of long centers takes up to the CU's LDS in one workgroup
        const size_t cu = prop.maxSharedMemoryPerMultiProcessor;
        if (cu > ctx->lds_max &&
            hipFuncSetAttribute((const void *)hk::rows_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)cu) ==
                hipSuccess)
            ctx->lds_cu = cu;
        else
            ctx->lds_cu = ctx->lds_max;
        (void)hipGetLastError();
    }
    if (hipHostMalloc((void **)&ctx->flag_host, 64, hipHostMallocDefault) != hipSuccess) {
        halign_ctx_destroy(ctx);
        return fail(HALIGN_E_DEVICE, "pinned allocation");
    }
    // the width mailbox; without it the width comes back by a copy and a
    // stream synchronisation
    if (hipHostMalloc((void **)&ctx->mail_host, 64, hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess) {
        ctx->mail_host[0] = ctx->mail_host[1] = 0;
        if (hipHostGetDevicePointer((void **)&ctx->mail_dev, ctx->mail_host, 0) != hipSuccess) ctx->mail_dev = nullptr;
    } else {
        ctx->mail_host = nullptr;
        (void)hipGetLastError();
    }
    if (hipEventCreateWithFlags(&ctx->ev_stage, hipEventDisableTiming) != hipSuccess) {
        halign_ctx_destroy(ctx);
        return fail(HALIGN_E_DEVICE, "event create");
    }
    eval_contexts(device, 1);
    ctx->counted = true;
    *out = ctx;
    return HALIGN_OK;
}

void halign_ctx_destroy(halign_ctx *ctx) {
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    if (ctx->counted) eval_contexts(ctx->device, -1);
    (void)hipDeviceSynchronize();
    graph_drop(ctx);
    if (ctx->cap_stream) (void)hipStreamDestroy(ctx->cap_stream);
    if (ctx->aux_stream) (void)hipStreamDestroy(ctx->aux_stream);
    for (DevBuf *b : {&ctx->codes, &ctx->bound, &ctx->plan, &ctx->counter, &ctx->pairbuf, &ctx->msabuf, &ctx->spbuf,
                      &ctx->sbuf, &ctx->histbuf, &ctx->nuctab, &ctx->nucscr, &ctx->nucdp, &ctx->rowck,
                      &ctx->njrows, &ctx->njD, &ctx->njS, &ctx->njacc, &ctx->njB, &ctx->njF})
        if (b->p) (void)hipFree(b->p);
    for (DevBuf &b : ctx->mlp)
        if (b.p) (void)hipFree(b.p);
    for (HostBuf *b : {&ctx->stage, &ctx->njhost, &ctx->njout})
        if (b->p) (void)hipHostFree(b->p);
    if (ctx->ev_nj) (void)hipEventDestroy(ctx->ev_nj);
    if (ctx->flag_host) (void)hipHostFree(ctx->flag_host);
    if (ctx->mail_host) (void)hipHostFree(ctx->mail_host);
    for (auto &t : ctx->tev)
        for (auto &e : t) (void)hipEventDestroy(e);
    if (ctx->ev_stage) (void)hipEventDestroy(ctx->ev_stage);
    delete ctx;
}

int halign_ctx_workspace_bytes(const halign_ctx *ctx, size_t *bytes_host) {
    if (!ctx || !bytes_host) return fail(HALIGN_E_INVALID, "NULL argument");
    *bytes_host = ctx->codes.cap + ctx->bound.cap + ctx->plan.cap + ctx->pairbuf.cap + ctx->msabuf.cap;
    return HALIGN_OK;
}

int halign_ctx_last_timings(halign_ctx *ctx, float *ms_host) {
    if (!ctx || !ms_host) return fail(HALIGN_E_INVALID, "NULL argument");
    RCHK(tev_sum(ctx, &ms_host[0], &ms_host[1]));
    ms_host[2] = ms_host[0] + ms_host[1];
    return HALIGN_OK;
}

int halign_ctx_last_stats(const halign_ctx *ctx, int64_t *stats_host) {
    if (!ctx || !stats_host) return fail(HALIGN_E_INVALID, "NULL argument");
    for (int i = 0; i < 4; ++i) stats_host[i] = ctx->last_stats[i];
    return HALIGN_OK;
}

int halign_ctx_set_graph(halign_ctx *ctx, int enable) {
    if (!ctx) return fail(HALIGN_E_INVALID, "NULL ctx");
    ctx->use_graph = enable != 0;
    if (!enable) graph_drop(ctx);
    return HALIGN_OK;
}

int halign_ctx_graph_launches(const halign_ctx *ctx, int64_t *n_host) {
    if (!ctx || !n_host) return fail(HALIGN_E_INVALID, "NULL argument");
    *n_host = ctx->graph_launches;
    return HALIGN_OK;
}

int halign_ctx_set_prejudge(halign_ctx *ctx, int candidates, int partners) {
    if (!ctx || candidates < 0 || candidates > 256 || partners < 0) return fail(HALIGN_E_INVALID, "bad arguments");
    ctx->prejudge_cand = candidates;
    ctx->prejudge_part = partners;
    return HALIGN_OK;
}

int halign_ctx_set_autotune(halign_ctx *ctx, int enable) {
    if (!ctx) return fail(HALIGN_E_INVALID, "NULL ctx");
    ctx->autotune = enable != 0;
    return HALIGN_OK;
}

int halign_ctx_last_plan(const halign_ctx *ctx, int32_t *plan_host) {
    if (!ctx || !plan_host) return fail(HALIGN_E_INVALID, "NULL argument");
    for (int i = 0; i < 5; ++i) plan_host[i] = ctx->last_tune[i];
    return HALIGN_OK;
}

// Failure injection (declared in halign.h): chunk `c` of the next
// halign_sw_batch fails before its launch.
int halign_debug_fail_chunk(halign_ctx *ctx, int c) {
    if (!ctx) return fail(HALIGN_E_INVALID, "NULL ctx");
    ctx->fault_chunk = c;
    return HALIGN_OK;
}

int halign_encode(const uint8_t *ascii, int64_t len, uint8_t *codes, void *stream) {
    static const char kAlpha[] = "ARNDCQEGHILKMFPSTWYVBZX*";
    if (len < 0 || (len > 0 && (!ascii || !codes))) return fail(HALIGN_E_INVALID, "bad arguments");
    if (len == 0) return HALIGN_OK;
    static uint8_t *dtab = nullptr;
    static int dtab_dev = -1;
    int dev = 0;
    HCHK(hipGetDevice(&dev));
    if (!dtab || dtab_dev != dev) {
        uint8_t tab[256];
        for (int x = 0; x < 256; ++x) tab[x] = 22;  // X
        for (int x = 0; x < 24; ++x) {
            tab[(uint8_t)kAlpha[x]] = (uint8_t)x;
            if (kAlpha[x] >= 'A' && kAlpha[x] <= 'Z') tab[(uint8_t)(kAlpha[x] - 'A' + 'a')] = (uint8_t)x;
        }
        tab['U'] = tab['u'] = 4;   // C
        tab['O'] = tab['o'] = 11;  // K
        uint8_t *p = nullptr;
        HCHK(hipMalloc(&p, 256));
        HCHK(hipMemcpy(p, tab, 256, hipMemcpyHostToDevice));
        dtab = p;
        dtab_dev = dev;
    }
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(hk::encode_kernel, dim3(grid_for(len, 256, 8192)), dim3(256), 0, st, ascii, len, codes,
                       (const uint8_t *)dtab);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

}  // extern "C"

// The launch sequence of halign_sw_batch (validation, plan, forward, walk).
static int sw_batch_body(halign_ctx *ctx, const halign_scoring *sc, const uint8_t *center, int32_t m,
                          const halign_seqs *seqs, uint32_t flags, int32_t *score, int32_t *cells, uint16_t *ins,
                          uint32_t *aligned, void *stream, int32_t *G = nullptr, int gskip = -1,
                          int longest = -1, bool fetch = true) {
    if (!ctx) return fail(HALIGN_E_INVALID, "ctx is NULL");
    if (longest < 0) {   // halign_msa has checked both already
        RCHK(check_scoring(sc));
        RCHK(check_seqs(seqs, &longest));
    }
    if (m <= 0 || !center) return fail(HALIGN_E_INVALID, "empty center");
    if (m >= 65536) return fail(HALIGN_E_UNSUPPORTED, "center length %d >= 65536", m);
    if (!score && seqs->n > 0) return fail(HALIGN_E_INVALID, "score is NULL");
    const bool tb = (flags & HALIGN_TRACEBACK) != 0;
    if (tb && (!cells || !ins || !aligned)) return fail(HALIGN_E_INVALID, "traceback needs cells, ins, aligned");
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    const int N = seqs->n;
    if (N == 0) return HALIGN_OK;
    Scoring S;
    const bool want_tune = ctx->autotune && (flags & (3u << 4)) == HALIGN_ROUTE_AUTO;
    hk::PrepArgs pa{};
    RCHK(upload_matrix(ctx, sc, st, &S, want_tune ? nullptr : &pa));   // (the tuner runs before)
    // endcells: needed by the walk, or to fill cells in score-only mode
    const bool endc = tb || cells != nullptr;
    RCHK(grow(ctx, ctx->pairbuf, (size_t)N * 8 + 256));
    int32_t *endcell = (int32_t *)ctx->pairbuf.p;
    hmark(ctx, "upload");
    const bool graph_call = (flags & HALIGN_GRAPH) != 0;   // planned on the host
    Tune tune;
    if (want_tune) {
        BatchOut tout{score, cells, endcell, ins, aligned};
        bool ran = false;
        RCHK(autotune(ctx, S, center, m, seqs, tb, endc, tout, graph_call ? -1 : longest, st, &tune, &ran));
        if (ran) RCHK(stage_begin(ctx));   // the tuner's runs have synchronised
    }
    for (auto &v : ctx->last_stats) v = 0;
    hmark(ctx, "tune");
    // the code check and the zeroing of the outputs go in before the host
    // plans the batch, so these small kernels run while the host works (the
    // forward kernels read codes masked to 5 bits, the check is read after the
    // batch, and the outputs are first written by the walk); with them the matrix
    // and the device planner's count of the pairs by length
    const bool count = !graph_call && N >= kDevPlanMin && longest < hk::kPrepHistMax;
    auto prep = [&]() -> int {
        if (tb) {
            // ins (as 32-bit words; an odd trailing uint16 on its own), aligned and G zeroed
            const int64_t nins = (int64_t)N * (m + 1);
            pa.z[0] = reinterpret_cast<uint32_t *>(ins);
            pa.nz[0] = nins / 2;
            pa.z[1] = aligned;
            pa.nz[1] = (int64_t)N * ((m + 31) / 32);
            pa.z[2] = reinterpret_cast<uint32_t *>(G);
            pa.nz[2] = G ? (int64_t)m + 1 : 0;
            pa.tail16 = (nins & 1) ? ins + (nins - 1) : nullptr;
        }
        if (count) {
            RCHK(grow(ctx, ctx->histbuf, 4 * (size_t)kHistParts * hk::kPrepHistMax));
            pa.off = seqs->offsets;
            pa.np = N;
            pa.maxlen = longest;
            pa.hwgs = kHistParts;
            pa.hpart = (int32_t *)ctx->histbuf.p;
        }
        RCHK(validate_codes(ctx, sc->alphabet, seqs->residues, seqs->offsets_host[N], center, m, st, pa));
        return HALIGN_OK;
    };
    BatchOut out{score, cells, endcell, ins, aligned};
    if (tb && G) {
        out.G = G;
        out.gskip = gskip;
    }
    RCHK(prep());
    hmark(ctx, "prep");
    // Routing by pair length: when the batch as a whole runs one pair per lane
    // (the route the caller did not force), pairs longer than kLongPair
    // residues run on the wavefront kernel, one pair per stream, in a launch
    // of their own; the rest keep the strip kernel.  Both write the same
    // outputs, each at its own pair ids.
    const int route = tune.route >= 0 ? tune.route : route_of(flags, sc, m, seqs, tb, longest);
    const int64_t *oh = seqs->offsets_host;
    const bool split = route == kRouteInter && (flags & (3u << 4)) == HALIGN_ROUTE_AUTO;
    int nlong = 0;
    if (split)
        for (int k = 0; k < N; ++k) nlong += oh[k + 1] - oh[k] > kLongPair;
    if (nlong == 0) {
        RCHK(run_batch(ctx, S, center, m, seqs, nullptr, N, tb, endc, route, out, st, tune,
                       graph_call ? -1 : longest, count));
    } else {
        // long pairs first in the id list, then the rest
        std::vector<int32_t> &ids = ctx->h_split;
        ids.resize(N);
        int a = 0, b = nlong;
        for (int k = 0; k < N; ++k) ids[oh[k + 1] - oh[k] > kLongPair ? a++ : b++] = k;
        RCHK(run_batch(ctx, S, center, m, seqs, ids.data(), nlong, tb, endc, kRouteIntra, out, st));
        RCHK(run_batch(ctx, S, center, m, seqs, ids.data() + nlong, N - nlong, tb, endc, route, out, st, tune));
    }
    ctx->last_tune = {tune.route, tune.R, tune.smul, tune.LS > 0 ? tune.LS : 64, ctx->last_pk};
    if (!tb && cells && ctx->last_stats[2] != kRouteIntra) {
        // score-only with cells, one pair per lane: report the end cell as (0, 0, i1, j1)
        hipLaunchKernelGGL(hk::endcell_to_cells_kernel, dim3(grid_for(N, 256)), dim3(256), 0, st,
                           (const int32_t *)endcell, N, cells);
        HCHK(hipGetLastError());
    }
    if (fetch) RCHK(flag_fetch(ctx, st));
    return HALIGN_OK;
}

namespace {

// FNV-1a over 8-byte words (then the tail bytes)
uint64_t fnv(uint64_t h, const void *p, size_t n) {
    const uint8_t *b = (const uint8_t *)p;
    size_t i = 0;
    for (; i + 8 <= n; i += 8) {
        uint64_t w;
        memcpy(&w, b + i, 8);
        h ^= w;
        h *= 0x100000001b3ull;
        h ^= h >> 29;
    }
    for (; i < n; ++i) { h ^= b[i]; h *= 0x100000001b3ull; }
    return h;
}

}  // namespace

// halign_sw_batch without the final synchronisation: the code check is left
// pending for the caller's next synchronisation point (validate_check).
// With HALIGN_GRAPH the launch sequence is captured once into a hipGraph that
// owns its scratch and plan buffers, and replayed while the call's arguments
// (pointers, sizes, offsets, scoring) stay the same.
static int sw_batch_async(halign_ctx *ctx, const halign_scoring *sc, const uint8_t *center, int32_t m,
                          const halign_seqs *seqs, uint32_t flags, int32_t *score, int32_t *cells, uint16_t *ins,
                          uint32_t *aligned, void *stream, int32_t *G = nullptr, int gskip = -1,
                          int longest = -1, bool fetch = true) {
    if (!(flags & HALIGN_GRAPH))
        return sw_batch_body(ctx, sc, center, m, seqs, flags, score, cells, ins, aligned, stream, G, gskip, longest,
                             fetch);
    if (!ctx || !sc || !seqs || !sc->matrix_host || !seqs->offsets_host)
        return sw_batch_body(ctx, sc, center, m, seqs, flags, score, cells, ins, aligned, stream, G, gskip);
    hipStream_t st = (hipStream_t)stream;
    uint64_t key = 0xcbf29ce484222325ull;
    const void *ptrs[8] = {center, seqs->residues, seqs->offsets, score, cells, ins, aligned, G};
    key = fnv(key, ptrs, sizeof ptrs);
    const int32_t ints[8] = {m, seqs->n, (int32_t)flags, sc->alphabet, sc->gap_open, sc->gap_extend, ctx->autotune,
                             gskip};
    key = fnv(key, ints, sizeof ints);
    if (sc->alphabet > 0 && sc->alphabet <= 32)
        key = fnv(key, sc->matrix_host, (size_t)sc->alphabet * sc->alphabet);
    if (seqs->n >= 0) key = fnv(key, seqs->offsets_host, sizeof(int64_t) * ((size_t)seqs->n + 1));
    if (ctx->gent.exec && ctx->gent.key == key) {
        HCHK(hipSetDevice(ctx->device));
        RCHK(stage_begin(ctx));
        std::array<hipEvent_t, 3> *tv = nullptr;
        RCHK(tev_next(ctx, &tv));
        RCHK(record(ctx, (*tv)[0], st));
        HCHK(hipGraphLaunch(ctx->gent.exec, st));
        RCHK(record(ctx, (*tv)[1], st));
        RCHK(record(ctx, (*tv)[2], st));
        ctx->flag_alpha = sc->alphabet;   // the graph copies the code check into flag_host
        ctx->check_tag = 0;               // with tag 0
        ctx->graph_launches++;
        return HALIGN_OK;
    }
    // first call: run it, then capture the same sequence for later calls
    RCHK(sw_batch_body(ctx, sc, center, m, seqs, flags, score, cells, ins, aligned, stream, G, gskip));
    // the captured run writes its plans into the stage from its start again:
    // the copies of the run above must have read it first
    RCHK(stage_wait(ctx));
    const int pending = ctx->flag_alpha;
    const uint32_t pending_tag = ctx->check_tag;
    graph_drop(ctx);
    if (!ctx->cap_stream) HCHK(hipStreamCreateWithFlags(&ctx->cap_stream, hipStreamNonBlocking));
    HCHK(hipStreamBeginCapture(ctx->cap_stream, hipStreamCaptureModeRelaxed));
    ctx->capturing = true;
    const int rc = sw_batch_body(ctx, sc, center, m, seqs, flags, score, cells, ins, aligned, ctx->cap_stream, G,
                                 gskip);
    ctx->capturing = false;
    hipGraph_t g = nullptr;
    const hipError_t ec = hipStreamEndCapture(ctx->cap_stream, &g);
    ctx->flag_alpha = pending;
    ctx->check_tag = pending_tag;
    if (rc != HALIGN_OK) {
        if (g) (void)hipGraphDestroy(g);
        return rc;
    }
    if (ec != hipSuccess) return fail(HALIGN_E_DEVICE, "graph capture failed: %s", hipGetErrorString(ec));
    hipGraphExec_t ex = nullptr;
    if (hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) != hipSuccess) {
        (void)hipGraphDestroy(g);
        return fail(HALIGN_E_DEVICE, "graph instantiation failed");
    }
    // the graph keeps the buffers it references; the ctx gets fresh ones later
    auto &e = ctx->gent;
    e.key = key;
    e.graph = g;
    e.exec = ex;
    std::swap(e.plan, ctx->plan);
    std::swap(e.codes, ctx->codes);
    std::swap(e.sbuf, ctx->sbuf);
    std::swap(e.bound, ctx->bound);
    std::swap(e.counter, ctx->counter);
    std::swap(e.pairbuf, ctx->pairbuf);
    std::swap(e.spbuf, ctx->spbuf);
    std::swap(e.stage, ctx->stage);
    ctx->stage_pending = false;
    return HALIGN_OK;
}

extern "C" {

int halign_sw_batch(halign_ctx *ctx, const halign_scoring *sc, const uint8_t *center, int32_t m,
                    const halign_seqs *seqs, uint32_t flags, int32_t *score, int32_t *cells, uint16_t *ins,
                    uint32_t *aligned, void *stream) {
    const int rc = sw_batch_async(ctx, sc, center, m, seqs, flags, score, cells, ins, aligned, stream);
    if (rc != HALIGN_OK) {
        if (ctx) RCHK(stage_close(ctx, (hipStream_t)stream));
        return rc;
    }
    if (ctx->flag_alpha) {
        HCHK(hipStreamSynchronize((hipStream_t)stream));
        ctx->stage_pending = false;
        RCHK(validate_check(ctx));
    }
    return HALIGN_OK;
}

}  // extern "C"

static int emit_rows(halign_ctx *ctx, const halign_seqs *seqs, int32_t m, const uint16_t *ins,
                     const uint32_t *aligned, const int32_t *G, const int64_t *col, int64_t width, uint8_t *msa,
                     int longest, hipStream_t st);

// Spin until the mailbox holds seq or a later one (a kernel's release store, after its other
// words); now and then ask the stream whether it failed or finished.
static int mail_wait(halign_ctx *ctx, int64_t seq, hipStream_t st) {
    volatile int64_t *mb = ctx->mail_host;
    for (uint64_t it = 1;; ++it) {
        if (mb[1] >= seq) break;
        if ((it & 4095) == 0) {
            const hipError_t q = hipStreamQuery(st);
            if (q == hipSuccess) {
                if (mb[1] >= seq) break;
                return fail(HALIGN_E_DEVICE, "the stream finished without its message");
            }
            if (q != hipErrorNotReady) return fail(HALIGN_E_DEVICE, "%s", hipGetErrorString(q));
        }
    }
    __atomic_thread_fence(__ATOMIC_ACQUIRE);
    return HALIGN_OK;
}

// col[p] = sum_{q<p} (G[q] + 1) and the MSA width (copied to the host and
// synchronised when width_host is given).
// check: the code check's flag comes to flag_host with the width.
static int merge_offsets(halign_ctx *ctx, const int32_t *G, int m1, int64_t *col, int64_t *width_host,
                         hipStream_t st, bool check = false) {
    RCHK(grow(ctx, ctx->spbuf, 4096));
    int64_t *dwidth = (int64_t *)((char *)ctx->spbuf.p + 2048);
    const bool mail = width_host && ctx->mail_dev && !ctx->capturing;
    const int64_t seq = mail ? ++ctx->mail_seq : 0;
    hipLaunchKernelGGL(hk::merge_scan_kernel, dim3(1), dim3(1024), 0, st, G, m1, col, dwidth,
                       mail ? ctx->mail_dev : nullptr, seq,
                       check ? (const uint32_t *)ctx->counter.p + 8 : nullptr);
    HCHK(hipGetLastError());
    if (mail) {
        RCHK(mail_wait(ctx, seq, st));
        *width_host = ctx->mail_host[0];
        if (check) *ctx->flag_host = (int)ctx->mail_host[2];
    } else if (width_host) {
        if (check) RCHK(flag_fetch(ctx, st));
        HCHK(hipMemcpyAsync(width_host, dwidth, 8, hipMemcpyDeviceToHost, st));
        HCHK(hipStreamSynchronize(st));
    }
    return HALIGN_OK;
}

extern "C" {

int halign_merge(halign_ctx *ctx, const uint16_t *ins, int32_t n, int32_t m, int32_t *G, int64_t *col,
                 int64_t *width_host, void *stream) {
    if (!ctx || !G || !col || m < 0 || n < 0 || (n > 0 && !ins)) return fail(HALIGN_E_INVALID, "bad arguments");
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    const int m1 = m + 1;
    RCHK(launch_fill((uint32_t *)G, 0u, m1, st));
    if (n > 0) {
        dim3 grid((m1 + 255) / 256, (n + hk::kMergeRows - 1) / hk::kMergeRows);
        if (grid.y > 65535) {
            // fold rows: launch in slices of 65535 * kMergeRows rows
            for (int64_t r0 = 0; r0 < n; r0 += (int64_t)65535 * hk::kMergeRows) {
                const int rn = (int)std::min<int64_t>(n - r0, (int64_t)65535 * hk::kMergeRows);
                dim3 g2((m1 + 255) / 256, (rn + hk::kMergeRows - 1) / hk::kMergeRows);
                hipLaunchKernelGGL(hk::merge_max_kernel, g2, dim3(256), 0, st, ins + r0 * m1, rn, m1, G);
            }
        } else {
            hipLaunchKernelGGL(hk::merge_max_kernel, grid, dim3(256), 0, st, ins, n, m1, G);
        }
        HCHK(hipGetLastError());
    }
    return merge_offsets(ctx, G, m1, col, width_host, st);
}

int halign_emit_rows(halign_ctx *ctx, const halign_seqs *seqs, int32_t m, const uint16_t *ins,
                     const uint32_t *aligned, const int32_t *G, const int64_t *col, int64_t width, uint8_t *msa,
                     void *stream) {
    if (!ctx || !seqs || m < 0 || width < m || (seqs->n > 0 && (!ins || !aligned || !G || !col || !msa)))
        return fail(HALIGN_E_INVALID, "bad arguments");
    int longest = 0;
    RCHK(check_seqs(seqs, &longest));
    HCHK(hipSetDevice(ctx->device));
    return emit_rows(ctx, seqs, m, ins, aligned, G, col, width, msa, longest, (hipStream_t)stream);
}

}  // extern "C"

// halign_emit_rows for checked arguments (longest: the longest sequence)
static int emit_rows(halign_ctx *ctx, const halign_seqs *seqs, int32_t m, const uint16_t *ins,
                     const uint32_t *aligned, const int32_t *G, const int64_t *col, int64_t width, uint8_t *msa,
                     int longest, hipStream_t st) {
    const int N = seqs->n;
    if (N == 0 || width == 0) return HALIGN_OK;
    const int m1 = m + 1, aw = (m + 31) / 32;
    // long centers: tasks of (row, 256 blocks) after a per-row count pass
    // (HALIGN_ROWS=chunk|lds picks a kernel for any center)
    bool chunk_rows = m1 > hk::kRowsChunkMinBlocks;
    if (const char *e = getenv("HALIGN_ROWS")) {
        if (!strcmp(e, "chunk")) chunk_rows = true;
        if (!strcmp(e, "lds")) chunk_rows = false;
    }
    if (chunk_rows) {
        const int nck = (m1 + hk::kRowChunk - 1) / hk::kRowChunk;
        RCHK(grow(ctx, ctx->rowck, 4 * (size_t)N * nck));
        int32_t *ck = (int32_t *)ctx->rowck.p;
        hk::RowsArgs ra{seqs->residues, seqs->offsets, N, m, ins, aligned, aw, G, col, width, 0, 0, 0, 0, msa};
        const int cgrid = std::max(1, std::min(N, ctx->num_cu * 8));
        hipLaunchKernelGGL(hk::rows_count_kernel, dim3(cgrid), dim3(512), 0, st, ra, ck, nck);
        HCHK(hipGetLastError());
        const int64_t ntask = (int64_t)N * nck;
        const int egrid = (int)std::max<int64_t>(1, std::min<int64_t>((ntask + 3) / 4, (int64_t)ctx->num_cu * 8));
        hipLaunchKernelGGL(hk::rows_chunk_kernel, dim3(egrid), dim3(256), 4 * hk::kRowWave, st, ra,
                           (const int32_t *)ck, nck);
        HCHK(hipGetLastError());
        return HALIGN_OK;
    }
    // LDS per wavefront: (m+1) insertion counts, the aligned bits, the residues
    // and a chunk of ch columns
    size_t lim = std::min<size_t>(ctx->lds_max, 64 * 1024);
    const int res_bytes = (std::min(longest, 4096) + 4 + 15) & ~15;   // of a row staged at most
    auto wave_bytes = [&](int ch) {
        return hk::rows_ins_bytes(m1) + hk::rows_bit_bytes(aw) + (size_t)res_bytes + 16 + (size_t)ch + 32;
    };
    int ch = (int)std::min<int64_t>(8192, (width + 15) & ~(int64_t)15), wpb = hk::kWaveRows;
    while (ch > 1024 && (size_t)wpb * wave_bytes(ch) > lim) ch = ((ch / 2) + 15) & ~15;
    while (wpb > 1 && (size_t)wpb * wave_bytes(ch) > lim) --wpb;
    if ((size_t)wpb * wave_bytes(ch) > lim && wave_bytes(ch) <= ctx->lds_cu) lim = ctx->lds_cu;   // long centers
    if ((size_t)wpb * wave_bytes(ch) > lim) return fail(HALIGN_E_UNSUPPORTED, "center length %d too long for row emission", m);
    if (width >= ((int64_t)1 << 31)) return fail(HALIGN_E_UNSUPPORTED, "MSA width %lld", (long long)width);
    const size_t gcb = 4 * (size_t)(m1 + 1);
    if ((size_t)wpb * wave_bytes(ch) + gcb > lim && (size_t)wpb * wave_bytes(ch) + gcb <= ctx->lds_cu)
        lim = ctx->lds_cu;   // the column table in LDS too
    const int gc_lds = (size_t)wpb * wave_bytes(ch) + gcb <= lim ? 1 : 0;
    hk::RowsArgs ra{seqs->residues, seqs->offsets, N, m, ins, aligned, aw, G, col, width, ch, (int)wave_bytes(ch),
                    res_bytes, gc_lds, msa};
    const size_t lds = (size_t)wpb * wave_bytes(ch) + (gc_lds ? gcb : 0);
    const int per_cu = std::max(1, std::min(8, (int)(ctx->lds_max / lds)));
    const int grid = std::max(1, std::min((N + wpb - 1) / wpb, ctx->num_cu * per_cu));
    hipLaunchKernelGGL(hk::rows_kernel, dim3(grid), dim3(64 * wpb), lds, st, ra);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

extern "C" {

// Center selection -----------------------------------------------------------
// The packed 16-bit score-only strip kernel applies when every H (max S times
// the longest sequence) plus go + ge stays below 15000, also plus 18 ge (its rows'
// offsets) below 16000, and go + ge <= 256.
// HALIGN_STRIP32=1 keeps the 32-bit kernel (tests of both paths).
static bool strip16_ok(const Scoring &S, const halign_seqs *sq) {
    const char *e = getenv("HALIGN_STRIP32");
    if (e && atoi(e) != 0) return false;
    int smax = 0;
    for (int x = 0; x < S.alpha * S.alpha; ++x) smax = std::max(smax, (int)S.hmat[x]);
    int64_t lmax = 0;
    for (int k = 0; k < sq->n; ++k) lmax = std::max(lmax, sq->offsets_host[k + 1] - sq->offsets_host[k]);
    const int64_t top = (int64_t)smax * lmax + S.goe;
    return S.goe <= 256 && S.ge <= 256 && top < 15000 && top + 18 * S.ge < 16000;
}

// Groups: 64 partners and one center (32-bit kernel) or two (16-bit kernel).
// Mode 1 (all pairs a < b of `perm`, in length order): the groups follow the
// closed-form triangular tilings of tiling.hpp, ngroups = tri_groups(N, 64) or
// pair_groups(N), with no per-group arrays.  Mode 2 (anchored groups): gcen, gb0
// and gslot list the groups; 16-bit, gcen and gslot hold the second centers
// and slots behind the first ones.
constexpr int64_t kGroupSlice = (int64_t)1 << 21;   // all-pairs groups per launch

static int run_groups(halign_ctx *ctx, const Scoring &S, const halign_seqs *sq, int mode, int64_t ngroups,
                      const std::vector<int32_t> &gcen, const std::vector<int32_t> &gb0,
                      const std::vector<int32_t> &perm, const std::vector<int32_t> &gslot, int64_t *sums,
                      int32_t *score, hipStream_t st, int nperm = -1, bool p16 = false) {
    if (p16 && (score || mode == 0)) return fail(HALIGN_E_INVALID, "16-bit strip kernel: score-only center selection");
    if (ngroups <= 0) return HALIGN_OK;
    const size_t ng2 = mode == 2 ? (size_t)ngroups : 1, nc2 = p16 ? 2 * ng2 : ng2;
    PlanBuilder pb;
    const size_t o_gcen = pb.add(4 * nc2), o_gb0 = pb.add(4 * ng2), o_perm = pb.add(4 * perm.size()),
                 o_gslot = pb.add(4 * nc2);
    // few groups for each of the resident wavefronts: run in order of falling cost
    // (by length buckets), so that they end together (9,600 groups of 1,500 proteins:
    // 21.2 ms against 22.4 from the last group down); from 65,536 on the order is worth under 1%
    const bool ordered = p16 && mode == 1 && ngroups < 65536 && !getenv("HALIGN_GROUP_SLICE");
    const size_t o_order = pb.add(ordered ? 4 * (size_t)ngroups : 0);
    char *hs = nullptr;
    RCHK(stage_host(ctx, pb.total, &hs));
    if (ordered) {
        const int64_t *off = sq->offsets_host;
        const int np = (int)perm.size();
        auto len = [&](int64_t pos) { return off[perm[pos] + 1] - off[perm[pos]]; };   // (longest last)
        const double top = (double)len(np - 1) * (double)len(np - 1) + 1;
        std::vector<int32_t> bucket(ngroups), first(1025, 0);
        for (int64_t g = 0; g < ngroups; ++g) {
            int64_t p0, b0;
            hk::pair_group(g, np, &p0, &b0);
            const double cost = (double)len(p0 + 1) * (double)len(std::min<int64_t>(np, b0 + 64) - 1);
            bucket[g] = 1023 - (int)(1024.0 * cost / top);
            ++first[bucket[g] + 1];
        }
        for (int q = 0; q < 1024; ++q) first[q + 1] += first[q];
        int32_t *order = (int32_t *)(hs + o_order);
        for (int64_t g = ngroups - 1; g >= 0; --g) order[first[bucket[g]]++] = (int32_t)g;
    }
    if (mode == 2) {
        memcpy(hs + o_gcen, gcen.data(), 4 * nc2);
        memcpy(hs + o_gb0, gb0.data(), 4 * ng2);
        memcpy(hs + o_gslot, gslot.data(), 4 * nc2);
    }
    memcpy(hs + o_perm, perm.data(), 4 * perm.size());
    char *dplan = nullptr;
    RCHK(plan_dev(ctx, pb.total, st, &dplan));
    HCHK(hipMemcpyAsync(dplan, hs, pb.total, hipMemcpyHostToDevice, st));
    stage_copied(ctx);
    RCHK(stage_close(ctx, st));
    int nmax_all = 0;
    const int64_t *oh = sq->offsets_host;
    for (int k = 0; k < sq->n; ++k) nmax_all = std::max(nmax_all, (int)(oh[k + 1] - oh[k]));
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(ngroups, (int64_t)ctx->num_cu * (p16 ? 12 : 16)));
    RCHK(grow(ctx, ctx->bound, (size_t)grid * 64 * strip_cols(nmax_all) * (p16 ? 9 : 8)));
    RCHK(grow(ctx, ctx->counter, 256));
    RCHK(launch_fill((uint32_t *)ctx->counter.p, 0u, 2, st));
    hk::InterArgs a{};
    a.mat = S.dmat;
    a.alpha = S.alpha;
    a.res = sq->residues;
    a.off = sq->offsets;
    a.mode = mode;
    a.gcen = (const int32_t *)(dplan + o_gcen);
    a.gb0 = (const int32_t *)(dplan + o_gb0);
    a.perm = (const int32_t *)(dplan + o_perm);
    a.nseq = nperm >= 0 ? nperm : sq->n;
    a.gslot = (const int32_t *)(dplan + o_gslot);
    a.gorder = ordered ? (const int32_t *)(dplan + o_order) : nullptr;
    a.gcen2 = a.gcen + ng2;
    a.gslot2 = a.gslot + ng2;
    a.sums = sums;
    a.ngroups = ngroups;
    a.ge = S.ge;
    a.goe = S.goe;
    a.counter = (unsigned long long *)ctx->counter.p;
    a.score = score;
    a.bound = (int2 *)ctx->bound.p;
    a.bstride = (int64_t)64 * strip_cols(nmax_all);
    ctx->last_stats[0] = 0;
    std::array<hipEvent_t, 3> *tv = nullptr;
    RCHK(tev_next(ctx, &tv));
    RCHK(record(ctx, (*tv)[0], st));
    // all pairs run in launches of at most kGroupSlice groups (a few seconds
    // each at the largest sets), so that no single kernel runs for minutes
    int64_t slice = mode == 1 ? kGroupSlice : ngroups;
    if (const char *e = getenv("HALIGN_GROUP_SLICE"))   // test knob: many small launches
        if (mode == 1 && atoll(e) > 0) slice = atoll(e);
    a.gtotal = ngroups;
    for (int64_t g0 = 0; g0 < ngroups; g0 += slice) {
        a.gfirst = g0;
        a.ngroups = std::min(slice, ngroups - g0);
        if (g0 > 0) RCHK(launch_fill((uint32_t *)ctx->counter.p, 0u, 2, st));
        if (p16) hipLaunchKernelGGL(hk::sw_inter16_kernel, dim3(grid), dim3(64), 0, st, a);
        else launch_inter(a, false, false, grid, st);
        HCHK(hipGetLastError());
        if (ctx->progress && ngroups > slice && !ctx->capturing) {
            HCHK(hipStreamSynchronize(st));
            fprintf(stderr, "halign: all-pairs groups %lld / %lld\n", (long long)(g0 + a.ngroups), (long long)ngroups);
        }
    }
    RCHK(record(ctx, (*tv)[1], st));
    RCHK(record(ctx, (*tv)[2], st));
    return HALIGN_OK;
}

static std::vector<int32_t> length_perm(const halign_seqs *sq) {
    std::vector<int32_t> perm(sq->n);
    std::iota(perm.begin(), perm.end(), 0);
    const int64_t *oh = sq->offsets_host;
    std::stable_sort(perm.begin(), perm.end(),
                     [&](int32_t x, int32_t y) { return (oh[x + 1] - oh[x]) < (oh[y + 1] - oh[y]); });
    return perm;
}

static int argmax_sums(halign_ctx *ctx, const int64_t *sums, const int32_t *cand_host, int ncand, int32_t *center_host,
                       hipStream_t st) {
    std::vector<int64_t> h(ncand);
    HCHK(hipMemcpyAsync(h.data(), sums, 8 * (size_t)ncand, hipMemcpyDeviceToHost, st));
    HCHK(hipStreamSynchronize(st));
    int best = 0;
    for (int q = 1; q < ncand; ++q) {
        const int cq = cand_host ? cand_host[q] : q, cb = cand_host ? cand_host[best] : best;
        if (h[q] > h[best] || (h[q] == h[best] && cq < cb)) best = q;
    }
    *center_host = cand_host ? cand_host[best] : best;
    (void)ctx;
    return HALIGN_OK;
}

int halign_exact_tiling(int64_t n, int32_t step, int64_t g, int64_t *ngroups_host, int64_t *center_pos_host,
                        int64_t *partner0_host) {
    const bool packed = step == HALIGN_TILING_PACKED;
    if (n < 0 || (step < 1 && !packed) || !ngroups_host) return fail(HALIGN_E_INVALID, "bad arguments");
    const int64_t ng = packed ? hk::pair_groups(n) : hk::tri_groups(n, step);
    *ngroups_host = ng;
    if (g < 0) return HALIGN_OK;
    if (g >= ng || !center_pos_host || !partner0_host) return fail(HALIGN_E_INVALID, "group %lld of %lld", (long long)g, (long long)ng);
    if (packed) hk::pair_group(g, n, center_pos_host, partner0_host);
    else hk::tri_group(g, n, step, center_pos_host, partner0_host);
    return HALIGN_OK;
}

int halign_center_exact(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs, int64_t *sums,
                        int32_t *center_host, void *stream) {
    if (!ctx || !sums) return fail(HALIGN_E_INVALID, "bad arguments");
    RCHK(check_scoring(sc));
    RCHK(check_seqs(seqs));
    const int N = seqs->n;
    if (N <= 0) return fail(HALIGN_E_INVALID, "empty set");
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    Scoring S;
    RCHK(upload_matrix(ctx, sc, st, &S));
    RCHK(validate_now(ctx, sc->alphabet, seqs->residues, seqs->offsets_host[N], nullptr, 0, st));
    RCHK(launch_fill((uint32_t *)sums, 0u, 2 * (int64_t)N, st));
    // all pairs a' < b' in length order: the longer sequence is the lane's,
    // the shorter one the group's center; the groups are numbered in closed
    // form (tiling.hpp), so the host holds O(N) plan data
    std::vector<int32_t> perm = length_perm(seqs), none;
    const bool p16 = strip16_ok(S, seqs);
    RCHK(run_groups(ctx, S, seqs, 1, p16 ? hk::pair_groups(N) : hk::tri_groups(N, 64), none, none, perm, none, sums, nullptr, st, -1, p16));
    if (center_host) RCHK(argmax_sums(ctx, sums, nullptr, N, center_host, st));
    return HALIGN_OK;
}

}  // extern "C"

// Sums of scores of candidates hc[q] against a partner list (NULL: every
// sequence), center = the candidate with the largest sum, ties to the lower
// sequence index.
static int judge_impl(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs,
                      const std::vector<int32_t> &hc, const int32_t *partners_host, int32_t npart, int64_t *sums,
                      int32_t *center_host, hipStream_t st) {
    const int N = seqs->n;
    const int ncand = (int)hc.size();
    for (int q = 0; q < ncand; ++q)
        if (hc[q] < 0 || hc[q] >= N) return fail(HALIGN_E_INVALID, "candidate %d out of range", hc[q]);
    Scoring S;
    RCHK(upload_matrix(ctx, sc, st, &S));
    RCHK(validate_now(ctx, sc->alphabet, seqs->residues, seqs->offsets_host[N], nullptr, 0, st));
    RCHK(launch_fill((uint32_t *)sums, 0u, 2 * (int64_t)ncand, st));
    std::vector<int32_t> perm, gcen, gb0, gslot;
    if (partners_host) {   // partners in length order, as for all sequences
        perm.assign(partners_host, partners_host + npart);
        const int64_t *oh = seqs->offsets_host;
        std::stable_sort(perm.begin(), perm.end(),
                         [&](int32_t x, int32_t y) { return (oh[x + 1] - oh[x]) < (oh[y + 1] - oh[y]); });
    } else {
        perm = length_perm(seqs);
    }
    const int np = (int)perm.size();
    const bool p16 = strip16_ok(S, seqs);
    const int cand_step = p16 ? 2 : 1;
    for (int q = 0; q < ncand; q += cand_step)
        for (int b = 0; b < np; b += 64) {
            gcen.push_back(hc[q]);
            gb0.push_back(b);
            gslot.push_back(q);
        }
    if (p16)   // the second centers
        for (int q = 1; q < ncand + 1; q += 2)
            for (int b = 0; b < np; b += 64) {
                gcen.push_back(q < ncand ? hc[q] : -1);
                gslot.push_back(std::min(q, ncand - 1));
            }
    RCHK(run_groups(ctx, S, seqs, 2, (int64_t)gb0.size(), gcen, gb0, perm, gslot, sums, nullptr, st, np, p16));
    if (center_host) RCHK(argmax_sums(ctx, sums, hc.data(), ncand, center_host, st));
    return HALIGN_OK;
}

extern "C" {

int halign_center_judge(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs, const int32_t *cand,
                        int32_t ncand, int64_t *sums, int32_t *center_host, void *stream) {
    if (!ctx || !sums || !cand || ncand <= 0) return fail(HALIGN_E_INVALID, "bad arguments");
    RCHK(check_scoring(sc));
    RCHK(check_seqs(seqs));
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    std::vector<int32_t> hc(ncand);
    HCHK(hipMemcpyAsync(hc.data(), cand, 4 * (size_t)ncand, hipMemcpyDeviceToHost, st));
    HCHK(hipStreamSynchronize(st));
    return judge_impl(ctx, sc, seqs, hc, nullptr, 0, sums, center_host, st);
}

int halign_center_judge_sample(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs,
                               const int32_t *cand, int32_t ncand, const int32_t *partners_host, int32_t npartners,
                               int64_t *sums, int32_t *center_host, void *stream) {
    if (!ctx || !sums || !cand || ncand <= 0 || npartners < 0 || (npartners > 0 && !partners_host))
        return fail(HALIGN_E_INVALID, "bad arguments");
    RCHK(check_scoring(sc));
    RCHK(check_seqs(seqs));
    const int N = seqs->n;
    for (int q = 0; q < npartners; ++q)
        if (partners_host[q] < 0 || partners_host[q] >= N) return fail(HALIGN_E_INVALID, "partner out of range");
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    std::vector<int32_t> hc(ncand);
    HCHK(hipMemcpyAsync(hc.data(), cand, 4 * (size_t)ncand, hipMemcpyDeviceToHost, st));
    HCHK(hipStreamSynchronize(st));
    return judge_impl(ctx, sc, seqs, hc, partners_host, npartners, sums, center_host, st);
}

int halign_sw_pairs(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs, const int32_t *anchors_host,
                    int32_t nanchors, const int32_t *partners_host, int32_t *score, void *stream) {
    if (!ctx || nanchors < 0 || (nanchors > 0 && (!anchors_host || !partners_host || !score)))
        return fail(HALIGN_E_INVALID, "bad arguments");
    RCHK(check_scoring(sc));
    RCHK(check_seqs(seqs));
    const int N = seqs->n;
    const int64_t np = (int64_t)nanchors * 64;
    for (int q = 0; q < nanchors; ++q)
        if (anchors_host[q] < 0 || anchors_host[q] >= N) return fail(HALIGN_E_INVALID, "anchor out of range");
    for (int64_t q = 0; q < np; ++q)
        if (partners_host[q] < 0 || partners_host[q] >= N) return fail(HALIGN_E_INVALID, "partner out of range");
    if (nanchors == 0) return HALIGN_OK;
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    Scoring S;
    RCHK(upload_matrix(ctx, sc, st, &S));
    RCHK(validate_now(ctx, sc->alphabet, seqs->residues, seqs->offsets_host[N], nullptr, 0, st));
    // group q: anchor q as the center, lanes = partners[64q .. 64q+63] (the
    // "perm" of the anchored mode), scores land at slot 64q + lane
    std::vector<int32_t> perm(partners_host, partners_host + np), gcen(anchors_host, anchors_host + nanchors),
        gb0(nanchors), gslot(nanchors);
    for (int q = 0; q < nanchors; ++q) {
        gb0[q] = q * 64;
        gslot[q] = q;
    }
    RCHK(grow(ctx, ctx->pairbuf, 16 * (size_t)nanchors + 256));
    int64_t *sums = (int64_t *)ctx->pairbuf.p;
    RCHK(launch_fill((uint32_t *)sums, 0u, 2 * (int64_t)nanchors, st));
    halign_seqs sq2 = *seqs;
    sq2.n = N;
    RCHK(run_groups(ctx, S, &sq2, 2, (int64_t)gcen.size(), gcen, gb0, perm, gslot, sums, score, st, (int)np));
    return HALIGN_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Allocation-free score-only batch: its scratch (matrix copy, work counter,
// strip boundary rows) is one static device array per GPU.  In host code the
// array's name only stands for the symbol; its device address on the current
// GPU comes from hipGetSymbolAddress, taken once per device and kept.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = HALIGN_NOALLOC_SCRATCH_BYTES;
constexpr size_t kScratchHead = 4096;   // matrix copy at 0, work counter at 2048, boundary rows after
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

struct ScratchSlot {
    void *ptr = nullptr;
    int num_cu = 0;
};
constexpr int kMaxDevices = 64;
ScratchSlot g_scratch[kMaxDevices];
std::mutex g_scratch_mu;

// the current device's copy of `scratch` (address and compute-unit count)
int scratch_of_device(int dev, ScratchSlot *out) {
    if (dev < 0 || dev >= kMaxDevices) return fail(HALIGN_E_UNSUPPORTED, "device %d", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    ScratchSlot &s = g_scratch[dev];
    if (!s.ptr) {
        void *p = nullptr;
        HCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        int cu = 0;
        HCHK(hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev));
        s.num_cu = std::max(1, cu);
        s.ptr = p;
    }
    *out = s;
    return HALIGN_OK;
}

}  // namespace

extern "C" {

int halign_sw_score_noalloc(const halign_scoring *sc, const uint8_t *center, int32_t m, const halign_seqs *seqs,
                            int32_t *score, int32_t *cells, void *stream) {
    RCHK(check_scoring(sc));
    RCHK(check_seqs(seqs));
    if (m <= 0 || !center) return fail(HALIGN_E_INVALID, "empty center");
    if (m >= 65536) return fail(HALIGN_E_UNSUPPORTED, "center length %d >= 65536", m);
    const int N = seqs->n;
    if (N == 0) return HALIGN_OK;
    if (!score) return fail(HALIGN_E_INVALID, "score is NULL");
    int dev = 0;
    HCHK(hipGetDevice(&dev));
    ScratchSlot sl;
    RCHK(scratch_of_device(dev, &sl));
    const int64_t *oh = seqs->offsets_host;
    int nmax_all = 0;
    for (int k = 0; k < N; ++k) nmax_all = std::max(nmax_all, (int)(oh[k + 1] - oh[k]));
    // boundary rows: 64 lanes x the longest sequence (whole prefetch blocks) per workgroup
    const int64_t bstride = (int64_t)64 * strip_cols(nmax_all);
    const size_t per_wg = (size_t)bstride * sizeof(int2);
    const size_t avail = kScratchBytes - kScratchHead;
    if (per_wg > avail)
        return fail(HALIGN_E_UNSUPPORTED,
                    "longest sequence %d needs %zu bytes of scratch per workgroup; the static scratch holds %zu",
                    nmax_all, per_wg, avail);
    const int64_t ngroups = ((int64_t)N + 63) / 64;
    const int grid = (int)std::max<int64_t>(
        1, std::min<int64_t>({ngroups, (int64_t)sl.num_cu * 16, (int64_t)(avail / per_wg)}));
    hipStream_t st = (hipStream_t)stream;
    unsigned char *base = (unsigned char *)sl.ptr;
    hk::MatrixArg mat{};
    memcpy(mat.v, sc->matrix_host, (size_t)sc->alphabet * sc->alphabet);
    hipLaunchKernelGGL(hk::matrix_copy_kernel, dim3(1), dim3(256), 0, st, mat, sc->alphabet * sc->alphabet,
                       (int8_t *)base);
    HCHK(hipGetLastError());
    // the work counter starts at zero on every call (the array keeps the last call's contents)
    RCHK(launch_fill((uint32_t *)(base + 2048), 0u, 2, st));
    hk::InterArgs a{};
    a.mat = (const int8_t *)base;
    a.alpha = sc->alphabet;
    a.center = center;
    a.m = m;
    a.res = seqs->residues;
    a.off = seqs->offsets;
    a.mode = 0;
    a.order = nullptr;
    a.gnmax = nullptr;
    a.nseq = N;
    a.ngroups = ngroups;
    a.ge = sc->gap_extend;
    a.goe = sc->gap_open + sc->gap_extend;
    a.counter = (unsigned long long *)(base + 2048);
    a.score = score;
    a.endcell = nullptr;
    a.cells4 = reinterpret_cast<int4 *>(cells);
    a.bound = (int2 *)(base + kScratchHead);
    a.bstride = bstride;
    launch_inter(a, false, cells != nullptr, grid, st);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

}  // extern "C"

// Column profile, *dbad raised to tag on a byte that is neither a residue code
// below alpha nor the gap.  Rows are split into slabs (at most kProfMaxSlab rows,
// for 16-bit partial counts); the slabs' counts meet in a second pass, not in
// atomics (many workgroups adding into the same profile line serialise).
// part: at least column_profile_part_bytes() bytes of device scratch.
static void column_profile_shape(int32_t n, int64_t width, int64_t *ncb, int64_t *nslab, int *slab) {
    if (n <= 0 || width <= 0) {   // nothing to count
        *ncb = *nslab = 0;
        *slab = 1;
        return;
    }
    *ncb = (width + hk::kProfCols - 1) / hk::kProfCols;
    // about two workgroups per CU, of at least 128 rows: each slab writes its
    // counts and the next pass reads them (20,000 x 4,030: 51 us a call with 32
    // slabs, 62 with 79, 61 with 20; 2,000 x 4,030: 33 with 16, 39 with 4)
    int64_t ns = std::max<int64_t>((n + hk::kProfMaxSlab - 1) / hk::kProfMaxSlab,
                                   std::min<int64_t>((512 + *ncb - 1) / *ncb, (n + 127) / 128));
    int sl = (int)((n + ns - 1) / std::max<int64_t>(ns, 1));
    if (const char *e = getenv("HALIGN_PROFILE_SLAB"))   // test knob: rows per slab
        if (atoi(e) > 0) sl = std::min(atoi(e), hk::kProfMaxSlab);
    *slab = std::max(sl, 1);
    *nslab = (n + *slab - 1) / *slab;
}

static size_t column_profile_part_bytes(int32_t n, int64_t width, int32_t alpha) {
    int64_t ncb, nslab;
    int slab;
    column_profile_shape(n, width, &ncb, &nslab, &slab);
    return (size_t)nslab * (size_t)width * (size_t)(alpha + 1) * 2;
}

// The slabs' counts into part (n > 0 and width > 0).
static int column_profile_launch(const uint8_t *msa, int32_t n, int64_t width, int32_t alpha, uint16_t *part,
                                 uint32_t *dbad, uint32_t tag, hipStream_t st, int *nslab_out) {
    int64_t ncb, nslab;
    int slab;
    column_profile_shape(n, width, &ncb, &nslab, &slab);
    *nslab_out = (int)nslab;
    if (ncb > 0x7fffffff || nslab > 65535) return fail(HALIGN_E_UNSUPPORTED, "%d x %lld MSA", n, (long long)width);
    hipLaunchKernelGGL(hk::colprof_kernel, dim3((unsigned)ncb, (unsigned)nslab), dim3(256),
                       (size_t)(alpha + 3) * 256 * 4, st, msa, n, width, alpha, slab, part, dbad, tag);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

// Scratch of the two evaluation calls, which have no context: a device buffer
// with its pinned mailbox, kept per device between calls while a context lives
// there (at most kEvalKeep bytes; allocating and freeing took 0.1 ms of a 0.13
// ms call).  Both calls synchronise before they return, so a buffer handed back
// is idle; a call that finds none kept (another thread holds it) allocates its
// own.
namespace {
constexpr size_t kEvalKeep = (size_t)64 << 20;
constexpr int kEvalDevices = 64;
// device: the flag word (raised to the call's tag, so it is never cleared), the
// workgroups' SP sums at 256, the slabs' counts at kEvalHead; pinned: a copy of
// the first kEvalHead bytes
constexpr size_t kEvalHead = 256 + (size_t)hk::kSpGroups * 16;
struct EvalBuf {
    char *dev = nullptr;
    size_t cap = 0;
    char *host = nullptr;
    uint32_t tag = 0;
};
std::mutex g_eval_mutex;
EvalBuf g_eval[kEvalDevices];
int g_eval_live[kEvalDevices];   // contexts on each device

void eval_free(EvalBuf &b) {
    if (b.dev) (void)hipFree(b.dev);
    if (b.host) (void)hipHostFree(b.host);
    b = EvalBuf();
}

int eval_take(size_t part_bytes, int *device, EvalBuf *out, hipStream_t st) {
    const size_t bytes = kEvalHead + part_bytes;
    HCHK(hipGetDevice(device));
    EvalBuf b;
    if (*device < kEvalDevices) {
        std::lock_guard<std::mutex> lk(g_eval_mutex);
        std::swap(b, g_eval[*device]);
    }
    if (b.cap < bytes) {
        eval_free(b);
        if (hipMalloc((void **)&b.dev, bytes) != hipSuccess) {
            (void)hipGetLastError();
            return fail(HALIGN_E_NOMEM, "device allocation of %zu bytes failed", bytes);
        }
        b.cap = bytes;
        if (hipHostMalloc((void **)&b.host, kEvalHead, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            b.host = nullptr;
            eval_free(b);
            return fail(HALIGN_E_DEVICE, "pinned allocation");
        }
        b.tag = 0;
    }
    if (b.tag == 0 || b.tag == 0xffffffffu) {   // a new buffer, or the tags are used up
        b.tag = 0;
        const int rc = launch_fill((uint32_t *)b.dev, 0u, 1, st);
        if (rc != HALIGN_OK) {
            eval_free(b);
            return rc;
        }
    }
    ++b.tag;
    *out = b;
    return HALIGN_OK;
}

void eval_give(int device, EvalBuf &b) {
    if (device < kEvalDevices && b.cap <= kEvalKeep) {
        std::lock_guard<std::mutex> lk(g_eval_mutex);
        if (g_eval_live[device] > 0 && !g_eval[device].dev) std::swap(b, g_eval[device]);
    }
    eval_free(b);
}

}  // namespace

// a context was created (+1) or destroyed (-1) on the device
static void eval_contexts(int device, int change) {
    if (device < 0 || device >= kEvalDevices) return;
    EvalBuf b;
    {
        std::lock_guard<std::mutex> lk(g_eval_mutex);
        g_eval_live[device] += change;
        if (g_eval_live[device] == 0) std::swap(b, g_eval[device]);
    }
    eval_free(b);
}

extern "C" {

int halign_column_profile(const uint8_t *msa, int32_t n, int64_t width, int32_t alphabet, int32_t *profile,
                          void *stream) {
    if (n < 0 || width < 0 || alphabet < 1 || alphabet > 32 || (width > 0 && !profile) ||
        (n > 0 && width > 0 && !msa))
        return fail(HALIGN_E_INVALID, "bad arguments");
    hipStream_t st = (hipStream_t)stream;
    int device = 0;
    EvalBuf b;
    RCHK(eval_take(column_profile_part_bytes(n, width, alphabet), &device, &b, st));
    const int64_t nelem = width * (alphabet + 1);
    auto body = [&]() -> int {
        if (n == 0 || width == 0) {
            RCHK(launch_fill((uint32_t *)profile, 0u, nelem, st));
            HCHK(hipStreamSynchronize(st));
            return HALIGN_OK;
        }
        uint16_t *part = (uint16_t *)(b.dev + kEvalHead);
        int nslab = 0;
        RCHK(column_profile_launch(msa, n, width, alphabet, part, (uint32_t *)b.dev, b.tag, st, &nslab));
        hipLaunchKernelGGL(hk::colprof_sum_kernel, dim3((unsigned)((nelem + 255) / 256)), dim3(256), 0, st,
                           (const uint16_t *)part, nslab, nelem, profile);
        HCHK(hipGetLastError());
        HCHK(hipMemcpyAsync(b.host, b.dev, 4, hipMemcpyDeviceToHost, st));
        HCHK(hipStreamSynchronize(st));
        if (*(const uint32_t *)b.host == b.tag)
            return fail(HALIGN_E_INVALID, "MSA byte neither a residue code below %d nor the gap", alphabet);
        return HALIGN_OK;
    };
    const int rc = body();
    if (rc != HALIGN_OK) (void)hipStreamSynchronize(st);
    eval_give(device, b);
    return rc;
}

int halign_sp_score(const halign_scoring *sc, const uint8_t *msa, int32_t n, int64_t width, int64_t *out_host,
                    void *stream) {
    RCHK(check_scoring(sc));
    if (!out_host || n < 0 || width < 0 || (n > 0 && width > 0 && !msa)) return fail(HALIGN_E_INVALID, "bad arguments");
    hipStream_t st = (hipStream_t)stream;
    const int alpha = sc->alphabet;
    if (n == 0 || width == 0) {
        HCHK(hipStreamSynchronize(st));
        out_host[0] = out_host[1] = 0;
        return HALIGN_OK;
    }
    int device = 0;
    EvalBuf b;
    RCHK(eval_take(column_profile_part_bytes(n, width, alpha), &device, &b, st));
    auto body = [&]() -> int {
        uint16_t *part = (uint16_t *)(b.dev + kEvalHead);
        int nslab = 0;
        RCHK(column_profile_launch(msa, n, width, alpha, part, (uint32_t *)b.dev, b.tag, st, &nslab));
        hk::SpMatrix mat;
        memcpy(mat.s, sc->matrix_host, (size_t)alpha * alpha);
        const int groups = (int)std::min<int64_t>(hk::kSpGroups, (width + hk::kSpCols - 1) / hk::kSpCols);
        hipLaunchKernelGGL(hk::sp_profile_kernel, dim3((unsigned)groups), dim3(256), 0, st, (const uint16_t *)part,
                           nslab, width, alpha, mat, sc->gap_extend, (int64_t *)(b.dev + 256));
        HCHK(hipGetLastError());
        HCHK(hipMemcpyAsync(b.host, b.dev, 256 + (size_t)groups * 16, hipMemcpyDeviceToHost, st));
        HCHK(hipStreamSynchronize(st));
        if (*(const uint32_t *)b.host == b.tag)
            return fail(HALIGN_E_INVALID, "MSA byte neither a residue code below %d nor the gap", alpha);
        const int64_t *h = (const int64_t *)(b.host + 256);
        out_host[0] = out_host[1] = 0;
        for (int q = 0; q < groups; ++q) {
            out_host[0] += h[2 * q];
            out_host[1] += h[2 * q + 1];
        }
        return HALIGN_OK;
    };
    const int rc = body();
    if (rc != HALIGN_OK) (void)hipStreamSynchronize(st);
    eval_give(device, b);
    return rc;
}

int halign_msa(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs, int32_t center,
               const halign_model *model, halign_alloc_fn alloc, void *user, uint8_t **msa, int64_t *width_host,
               int32_t *center_out_host, void *stream) {
    if (!ctx || !alloc || !msa || !width_host) return fail(HALIGN_E_INVALID, "bad arguments");
    ctx->hmarks.clear();
    hmark(ctx, "start");
    RCHK(check_scoring(sc));
    int longest = 0;
    RCHK(check_seqs(seqs, &longest));
    hmark(ctx, "checks");
    const int N = seqs->n;
    if (N <= 0) return fail(HALIGN_E_INVALID, "empty set");
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    int32_t c = center;
    if (center == HALIGN_CENTER_EXACT) {
        RCHK(grow(ctx, ctx->msabuf, 16 * (size_t)N + 256));
        RCHK(halign_center_exact(ctx, sc, seqs, (int64_t *)ctx->msabuf.p, &c, stream));
    } else if (center == HALIGN_CENTER_LEARNED) {
        if (!model) return fail(HALIGN_E_INVALID, "learned center needs a model");
        RCHK(halign_center_learned(ctx, sc, seqs, model, 16, nullptr, &c, stream));
    } else if (center < 0 || center >= N) {
        return fail(HALIGN_E_INVALID, "center %d out of range", center);
    }
    const int64_t *oh = seqs->offsets_host;
    const int m = (int)(oh[c + 1] - oh[c]);
    if (m <= 0) return fail(HALIGN_E_INVALID, "center sequence is empty");
    const int aw = (m + 31) / 32;
    // per-pair outputs in one workspace
    const size_t b_score = 4 * (size_t)N, b_cells = 16 * (size_t)N, b_ins = 2 * (size_t)N * (m + 1) + 4,
                 b_al = 4 * (size_t)N * aw, b_G = 4 * (size_t)(m + 1), b_col = 8 * (size_t)(m + 1);
    size_t o = 0;
    auto take = [&](size_t b) { size_t r = o; o = (o + b + 255) & ~size_t(255); return r; };
    const size_t o_score = take(b_score), o_cells = take(b_cells), o_ins = take(b_ins), o_al = take(b_al),
                 o_G = take(b_G), o_col = take(b_col);
    DevBuf &W = ctx->msabuf;
    RCHK(grow(ctx, W, o));
    char *wb = (char *)W.p;
    int32_t *score = (int32_t *)(wb + o_score);
    int32_t *cells = (int32_t *)(wb + o_cells);
    uint16_t *ins = (uint16_t *)(wb + o_ins);
    uint32_t *al = (uint32_t *)(wb + o_al);
    int32_t *G = (int32_t *)(wb + o_G);
    int64_t *col = (int64_t *)(wb + o_col);
    const uint8_t *cen = seqs->residues + oh[c];
    // the walk max-merges every pair's insertion counts into G (the center's own are all zero)
    // and leaves the center's own row; the code check's result comes with the
    // width (a captured batch copies it itself)
    const bool graph = ctx->use_graph != 0;
    const int rcb = sw_batch_async(ctx, sc, cen, m, seqs, HALIGN_TRACEBACK | (graph ? HALIGN_GRAPH : 0u), score, cells,
                                   ins, al, stream, G, c, longest, graph);
    int64_t width = 0;
    hmark(ctx, "batch");
    const int rcm = rcb != HALIGN_OK ? rcb : merge_offsets(ctx, G, m + 1, col, &width, st, !graph);   // synchronises
    if (rcm != HALIGN_OK) {
        RCHK(stage_close(ctx, st));
        return rcm;
    }
    ctx->stage_pending = false;
    hmark(ctx, "sync");
    RCHK(validate_check(ctx));
    uint8_t *out = (uint8_t *)alloc((size_t)N * (size_t)width, user);
    if (!out && width > 0) return fail(HALIGN_E_NOMEM, "allocator returned NULL for %lld bytes", (long long)(N * width));
    hmark(ctx, "alloc");
    RCHK(emit_rows(ctx, seqs, m, ins, al, G, col, width, out, longest, st));
    hmark(ctx, "rows");
    hmark_print(ctx);
    *msa = out;
    *width_host = width;
    if (center_out_host) *center_out_host = c;
    return HALIGN_OK;
}

}  // extern "C"

// ===========================================================================
// Learned center proposer
// ===========================================================================
namespace {

template <bool TA, bool TB, int EPI>
int gemm(const hk::GemmArgs &g, hipStream_t st) {
    if (g.M <= 0 || g.N <= 0) return HALIGN_OK;
    dim3 grid((g.N + 63) / 64, (g.M + 63) / 64);
    if (grid.y > 65535) return fail(HALIGN_E_UNSUPPORTED, "GEMM with %d rows", g.M);
    hipLaunchKernelGGL((hk::gemm_bf16_kernel<TA, TB, EPI>), grid, dim3(256), 0, st, g);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

// The pipelined product (packed B, rows of A 16-byte aligned).
template <int BM, int BN, int WM, int WN, bool TA, int EPI, int PF>
int gemm_tile(const hk::GemmArgs &g, hipStream_t st) {
    if (g.M <= 0) return HALIGN_OK;
    // epilogue 3 also writes the zero rows that pad its packed output
    const int rows = EPI == 3 ? (g.M + hk::kGK - 1) / hk::kGK * hk::kGK : g.M;
    const int mt = (rows + BM - 1) / BM, nt = g.N / BN;
    hipLaunchKernelGGL((hk::gemm_tile_kernel<BM, BN, WM, WN, TA, EPI, PF>), dim3((mt + 7) / 8 * 8 * nt),
                       dim3(64 * (BM / WM) * (BN / WN)), 0, st, g, mt, nt);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

// Whether the pipelined products may run: their 16-byte loads of A need
// aligned operands (the callers' pointers may have any alignment the element
// type allows), and their scratch `buf` must be there or be allocatable (not
// while `st` is being captured).
bool tile_ok(const DevBuf &buf, size_t bytes, hipStream_t st, std::initializer_list<const void *> ptrs) {
    for (const void *p : ptrs)
        if ((uintptr_t)p & 15) return false;
    if (bytes <= buf.cap) return true;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(st, &cs) == hipSuccess && cs == hipStreamCaptureStatusNone;
}

// fixed-order column sums of one or two rows x cols fp32 matrices (cols
// multiples of 64) into out
int colsum(halign_ctx *ctx, DevBuf &scratch, hk::ColsumArgs a, hipStream_t st) {
    const int nblk = std::max(1, (a.rows + hk::kColRows - 1) / hk::kColRows), cols = a.cols[0] + a.cols[1];
    RCHK(grow(ctx, scratch, (size_t)nblk * cols * 4 + 256));
    a.part[0] = (float *)scratch.p;
    a.part[1] = a.part[0] + (size_t)nblk * a.cols[0];
    if (a.rows > 0)
        hipLaunchKernelGGL(hk::colsum_partial_kernel, dim3(cols / 64, nblk), dim3(1024), 0, st, a);
    else
        RCHK(launch_fill((uint32_t *)scratch.p, 0u, cols, st));
    hipLaunchKernelGGL(hk::colsum_final_kernel, dim3((cols + 255) / 256), dim3(256), 0, st, a, nblk);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

uint64_t splitmix(uint64_t &s) {
    uint64_t z = (s += 0x9e3779b97f4a7c15ull);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

int check_model(const halign_model *md) {
    if (!md || !md->W1 || !md->b1 || !md->W2 || !md->b2) return fail(HALIGN_E_INVALID, "model pointers are NULL");
    return HALIGN_OK;
}

}  // namespace

extern "C" {

int halign_featurize(const halign_seqs *seqs, const int32_t *rows, int32_t nrows, uint16_t *X, void *stream) {
    if (!seqs || nrows < 0 || (nrows > 0 && !X)) return fail(HALIGN_E_INVALID, "bad arguments");
    RCHK(check_seqs(seqs));
    if (!rows && nrows > seqs->n) return fail(HALIGN_E_INVALID, "nrows > N");
    if (nrows == 0) return HALIGN_OK;
    hipLaunchKernelGGL(hk::featurize_kernel, dim3(nrows), dim3(256), 0, (hipStream_t)stream, seqs->residues,
                       seqs->offsets, rows, nrows, X);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

int halign_mlp_forward(halign_ctx *ctx, const halign_model *model, const uint16_t *X, int32_t nrows, float *Z,
                       uint16_t *Hb, float *E, void *stream) {
    if (!ctx || nrows < 0 || (nrows > 0 && (!X || !Hb || !E))) return fail(HALIGN_E_INVALID, "bad arguments");
    RCHK(check_model(model));
    if (nrows == 0) return HALIGN_OK;
    hipStream_t st = (hipStream_t)stream;
    hk::GemmArgs g1{};
    g1.A = X; g1.B = model->W1; g1.M = nrows; g1.N = hk::kHid; g1.K = hk::kFeat; g1.lda = hk::kFeat; g1.ldb = hk::kHid;
    g1.C = Z; g1.ldc = hk::kHid; g1.bias = model->b1; g1.Cb = Hb; g1.ldcb = hk::kHid;
    hk::GemmArgs g2{};
    g2.A = Hb; g2.B = model->W2; g2.M = nrows; g2.N = hk::kEmb; g2.K = hk::kHid; g2.lda = hk::kHid; g2.ldb = hk::kEmb;
    g2.C = E; g2.ldc = hk::kEmb; g2.bias = model->b2;
    const size_t b_p1 = (size_t)hk::kPackW1 * 16, b_p2 = (size_t)hk::kPackW2 * 16;
    if (!tile_ok(ctx->mlp[9], b_p1 + b_p2, st, {X, Hb})) {
        RCHK((gemm<false, false, 1>(g1, st)));
        return gemm<false, false, 0>(g2, st);
    }
    RCHK(grow(ctx, ctx->mlp[9], b_p1 + b_p2));
    uint16_t *P1 = (uint16_t *)ctx->mlp[9].p, *P2 = (uint16_t *)((char *)ctx->mlp[9].p + b_p1);
    hipLaunchKernelGGL(hk::pack_weights_kernel, dim3((hk::kPackW1 + hk::kPackW2 + 255) / 256), dim3(256), 0, st,
                       model->W1, model->W2, P1, P2);
    HCHK(hipGetLastError());
    g1.B = P1;
    g2.B = P2;
    // X . W1: the smallest tile that leaves at most one workgroup per CU (us,
    // K = 8000, N = 256): 2,048 rows 22 / 28 / 47 / 62 for the four tiles,
    // 4,096 rows 37 / 31 / 47 / 62, 8,192 rows 67 / 56 / 51 / 65, 16,384 rows
    // 169 / 144 / 129 / 100; a smaller tile reads W1 more often, a larger one
    // leaves CUs idle
    if ((nrows + 31) / 32 * 4 <= ctx->num_cu) RCHK((gemm_tile<32, 64, 32, 32, false, 1, 4>(g1, st)));
    else if ((nrows + 63) / 64 * 4 <= ctx->num_cu) RCHK((gemm_tile<64, 64, 32, 32, false, 1, 4>(g1, st)));
    else if ((nrows + 63) / 64 * 2 <= ctx->num_cu) RCHK((gemm_tile<64, 128, 32, 64, false, 1, 4>(g1, st)));
    else RCHK((gemm_tile<64, 256, 64, 64, false, 1, 4>(g1, st)));
    return gemm_tile<32, 32, 32, 32, false, 0, 2>(g2, st);
}

int halign_pair_loss(halign_ctx *ctx, const float *E, const float *target, int32_t npairs, float *dE,
                     float *loss_out, void *stream) {
    if (!ctx || npairs < 0 || (npairs > 0 && (!E || !target || !dE || !loss_out)))
        return fail(HALIGN_E_INVALID, "bad arguments");
    hipStream_t st = (hipStream_t)stream;
    RCHK(grow(ctx, ctx->mlp[0], (size_t)npairs * 4 + 512));
    float *sq = (float *)ctx->mlp[0].p;
    if (npairs > 0) {
        hipLaunchKernelGGL(hk::pair_loss_kernel, dim3((npairs + hk::kLossPairs - 1) / hk::kLossPairs), dim3(256), 0, st,
                           E, target, npairs, dE, sq);
        HCHK(hipGetLastError());
    }
    hipLaunchKernelGGL(hk::mean_kernel, dim3(1), dim3(256), 0, st, (const float *)sq, npairs, loss_out);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

int halign_pair_loss_grouped(halign_ctx *ctx, const float *E, const float *target, int32_t npairs, int32_t group,
                             float lam, float *dE, float *loss_out, void *stream) {
    if (group <= 0) return halign_pair_loss(ctx, E, target, npairs, dE, loss_out, stream);
    if (!ctx || npairs < 0 || group > 64 || npairs % group != 0 ||
        (npairs > 0 && (!E || !target || !dE || !loss_out)))
        return fail(HALIGN_E_INVALID, "bad arguments (1 <= group <= 64 dividing npairs)");
    hipStream_t st = (hipStream_t)stream;
    const int G = npairs / group;
    const size_t b_sq = ((size_t)npairs * 4 + 255) & ~size_t(255), b_g = ((size_t)G * 4 + 255) & ~size_t(255);
    RCHK(grow(ctx, ctx->mlp[0], b_sq + b_g + 512));
    float *sq = (float *)ctx->mlp[0].p;
    float *gsq = (float *)((char *)ctx->mlp[0].p + b_sq);
    if (G > 0) {
        hipLaunchKernelGGL(hk::pair_group_loss_kernel, dim3(G), dim3(64), 0, st, E, target, npairs, group, lam, dE,
                           sq, gsq);
        HCHK(hipGetLastError());
    }
    hipLaunchKernelGGL(hk::mean2_kernel, dim3(1), dim3(256), 0, st, (const float *)sq, npairs, (const float *)gsq, G,
                       lam, loss_out);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

int halign_mlp_backward(halign_ctx *ctx, const halign_model *model, const uint16_t *X, int32_t nrows, const float *Z,
                        const uint16_t *Hb, const float *dE, float *dW1, float *db1, float *dW2, float *db2,
                        void *stream) {
    if (!ctx || nrows < 0 || !dW1 || !db1 || !dW2 || !db2 || (nrows > 0 && (!X || !Z || !Hb || !dE)))
        return fail(HALIGN_E_INVALID, "bad arguments");
    RCHK(check_model(model));
    hipStream_t st = (hipStream_t)stream;
    auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
    const size_t rpad = ((size_t)nrows + 63) / 64 * 64;
    const size_t b_dEb = al((size_t)nrows * hk::kEmb * 2), b_dZ = al((size_t)nrows * hk::kHid * 4),
                 b_dZb = al(rpad * hk::kHid * 2), b_Pd = al(rpad * hk::kEmb * 2), b_P2t = al((size_t)hk::kPackW2T * 16);
    RCHK(grow(ctx, ctx->mlp[1], b_dEb + b_dZ + b_dZb + b_Pd + b_P2t));
    char *w = (char *)ctx->mlp[1].p;
    uint16_t *dEb = (uint16_t *)w, *dZb = (uint16_t *)(w + b_dEb + b_dZ), *Pd = (uint16_t *)(w + b_dEb + b_dZ + b_dZb),
             *P2t = (uint16_t *)(w + b_dEb + b_dZ + b_dZb + b_Pd);
    float *dZ = (float *)(w + b_dEb);
    // dW2 = Hb^T dEb, dZ = (dEb W2^T) * (Z > 0), dW1 = X^T dZb
    hk::GemmArgs a{}, b{}, c{};
    a.A = Hb; a.B = dEb; a.M = hk::kHid; a.N = hk::kEmb; a.K = nrows; a.lda = hk::kHid; a.ldb = hk::kEmb;
    a.C = dW2; a.ldc = hk::kEmb;
    b.A = dEb; b.B = model->W2; b.M = nrows; b.N = hk::kHid; b.K = hk::kEmb; b.lda = hk::kEmb; b.ldb = hk::kEmb;
    b.C = dZ; b.ldc = hk::kHid; b.Cb = dZb; b.ldcb = hk::kHid; b.Hpre = Z; b.ldh = hk::kHid;
    c.A = X; c.B = dZb; c.M = hk::kFeat; c.N = hk::kHid; c.K = nrows; c.lda = hk::kFeat; c.ldb = hk::kHid;
    c.C = dW1; c.ldc = hk::kHid;
    const bool tile = tile_ok(ctx->mlp[1], 0, st, {X, Hb});
    if (nrows == 0) {
        RCHK(launch_fill((uint32_t *)dW2, 0u, (int64_t)hk::kHid * hk::kEmb, st));
        RCHK(launch_fill((uint32_t *)dW1, 0u, (int64_t)hk::kFeat * hk::kHid, st));
    } else if (tile) {
        hipLaunchKernelGGL(hk::pack_backward_kernel, dim3((hk::pack_octets(nrows, hk::kEmb) + hk::kPackW2T + 255) / 256),
                           dim3(256), 0, st, dE, nrows, dEb, Pd, model->W2, P2t);
        HCHK(hipGetLastError());
        a.B = Pd;
        b.B = P2t;
        RCHK((gemm_tile<32, 32, 32, 32, true, 0, 2>(a, st)));
        RCHK((gemm_tile<32, 64, 32, 32, false, 3, 2>(b, st)));
        RCHK((gemm_tile<64, 128, 32, 64, true, 0, 4>(c, st)));
    } else {
        hipLaunchKernelGGL(hk::f32_to_bf16_kernel, dim3(grid_for((int64_t)nrows * hk::kEmb, 256, 4096)), dim3(256), 0,
                           st, dE, dEb, (int64_t)nrows * hk::kEmb);
        HCHK(hipGetLastError());
        RCHK((gemm<true, false, 0>(a, st)));
        RCHK((gemm<false, true, 2>(b, st)));
        RCHK((gemm<true, false, 0>(c, st)));
    }
    hk::ColsumArgs cs{};
    cs.A[0] = dE; cs.cols[0] = hk::kEmb; cs.out[0] = db2;
    cs.A[1] = dZ; cs.cols[1] = hk::kHid; cs.out[1] = db1;
    cs.rows = nrows;
    return colsum(ctx, ctx->mlp[2], cs, st);
}

int halign_f32_to_bf16(const float *src, uint16_t *dst, int64_t n, void *stream) {
    if (n < 0 || (n > 0 && (!src || !dst))) return fail(HALIGN_E_INVALID, "bad arguments");
    if (n == 0) return HALIGN_OK;
    hipLaunchKernelGGL(hk::f32_to_bf16_kernel, dim3(grid_for(n, 256, 8192)), dim3(256), 0, (hipStream_t)stream, src,
                       dst, n);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

int halign_adam_step(float *p, const float *g, float *m, float *v, uint16_t *pb, int64_t n, float lr, float beta1,
                     float beta2, float eps, int32_t t, void *stream) {
    if (n < 0 || t < 1 || (n > 0 && (!p || !g || !m || !v))) return fail(HALIGN_E_INVALID, "bad arguments");
    if (n == 0) return HALIGN_OK;
    const float c1 = 1.f - powf(beta1, (float)t), c2 = 1.f - powf(beta2, (float)t);
    hipLaunchKernelGGL(hk::adam_kernel, dim3(grid_for(n, 256, 8192)), dim3(256), 0, (hipStream_t)stream, p, g, m, v, pb,
                       n, lr, beta1, beta2, eps, c1, c2);
    HCHK(hipGetLastError());
    return HALIGN_OK;
}

int halign_topk_center(halign_ctx *ctx, const float *E, int32_t nrows, int32_t k, float *u, int32_t *top,
                       void *stream) {
    if (!ctx || !E || !u || !top || nrows <= 0 || k <= 0 || k > nrows || k > 256)
        return fail(HALIGN_E_INVALID, "bad arguments (1 <= k <= min(N, 256))");
    hipStream_t st = (hipStream_t)stream;
    RCHK(grow(ctx, ctx->mlp[3], 4096));
    float *S = (float *)ctx->mlp[3].p;
    hk::ColsumArgs cs{};
    cs.A[0] = E; cs.cols[0] = hk::kEmb; cs.out[0] = S; cs.rows = nrows;
    RCHK(colsum(ctx, ctx->mlp[2], cs, st));
    hipLaunchKernelGGL(hk::center_score_kernel, dim3((nrows + 255) / 256), dim3(256), 0, st, E, (const float *)S, nrows,
                       u);
    HCHK(hipGetLastError());
    // rounds of block top-k until one block holds everything
    int n = nrows;
    const float *val = u;
    const int32_t *idx = nullptr;
    int round = 0;
    for (;;) {
        const int nblk = (n + hk::kTopkChunk - 1) / hk::kTopkChunk;
        const size_t need = (size_t)nblk * k * 8 + 512;
        DevBuf &buf = ctx->mlp[4 + (round & 1)];
        RCHK(grow(ctx, buf, need));
        float *ov = (float *)buf.p;
        int32_t *oi = (int32_t *)((char *)buf.p + (((size_t)nblk * k * 4 + 255) & ~size_t(255)));
        hipLaunchKernelGGL(hk::topk_kernel, dim3(nblk), dim3(256), 0, st, val, idx, n, k, ov, oi);
        HCHK(hipGetLastError());
        if (nblk == 1) {
            HCHK(hipMemcpyAsync(top, oi, 4 * (size_t)k, hipMemcpyDeviceToDevice, st));
            break;
        }
        val = ov;
        idx = oi;
        n = nblk * k;
        ++round;
    }
    return HALIGN_OK;
}

int halign_train_proposer(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs,
                          const halign_train_opts *opts, const halign_params *pr, float *loss_host, void *stream) {
    if (!ctx || !opts || !pr || !pr->W1 || !pr->b1 || !pr->W2 || !pr->b2 || !pr->W1b || !pr->W2b)
        return fail(HALIGN_E_INVALID, "bad arguments");
    RCHK(check_scoring(sc));
    RCHK(check_seqs(seqs));
    const int N = seqs->n;
    if (N < 2 || opts->anchors <= 0 || opts->batch <= 0 || opts->epochs <= 0)
        return fail(HALIGN_E_INVALID, "need N >= 2 and positive anchors, batch, epochs");
    hipStream_t st = (hipStream_t)stream;
    HCHK(hipSetDevice(ctx->device));
    // training pairs: anchors with `partners` partners each (never the anchor
    // itself); the score kernel takes 64 partners per anchor, of which the
    // first `partners` are used
    uint64_t rs = opts->seed;
    const int A = opts->anchors;
    const int PA = (opts->partners > 0 && opts->partners < 64) ? opts->partners : 64;
    const int P = A * PA;
    std::vector<int32_t> anc(A), par((size_t)A * 64);
    for (int q = 0; q < A; ++q) anc[q] = (int32_t)(splitmix(rs) % (uint64_t)N);
    for (size_t q = 0; q < (size_t)A * 64; ++q) {
        int32_t b;
        do { b = (int32_t)(splitmix(rs) % (uint64_t)N); } while (b == anc[q / 64]);
        par[q] = b;
    }
    // with a group weight, a batch holds whole anchors (all PA partners of
    // each), and the loss adds the squared mean error of each anchor's pairs
    const bool grouped = opts->group_weight > 0.f;
    // scratch layout in mlp[6]: scores, targets, batch index lists, X_all
    const int B = grouped ? std::max(1, std::min(opts->batch, P) / PA) * PA : std::min(opts->batch, P);
    const int steps_per_epoch = P / B;
    const int nsteps = steps_per_epoch * opts->epochs;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t r = off; off = (off + bytes + 255) & ~size_t(255); return r; };
    const size_t o_score = take(4 * (size_t)A * 64), o_tgt = take(4 * (size_t)A * 64),
                 o_idx = take(4 * (size_t)nsteps * 2 * B),
                 o_tix = take(4 * (size_t)nsteps * B), o_tb = take(4 * (size_t)B), o_loss = take(4 * (size_t)nsteps),
                 o_X = take(2 * (size_t)N * hk::kFeat), o_Xb = take(2 * (size_t)2 * B * hk::kFeat),
                 o_Z = take(4 * (size_t)2 * B * hk::kHid), o_Hb = take(2 * (size_t)2 * B * hk::kHid),
                 o_E = take(4 * (size_t)2 * B * hk::kEmb), o_dE = take(4 * (size_t)2 * B * hk::kEmb),
                 o_g = take(4 * (size_t)(hk::kFeat * hk::kHid + hk::kHid + hk::kHid * hk::kEmb + hk::kEmb)),
                 o_m = take(4 * (size_t)(hk::kFeat * hk::kHid + hk::kHid + hk::kHid * hk::kEmb + hk::kEmb)),
                 o_v = take(4 * (size_t)(hk::kFeat * hk::kHid + hk::kHid + hk::kHid * hk::kEmb + hk::kEmb)),
                 o_e = take(4 * (size_t)(hk::kFeat * hk::kHid + hk::kHid + hk::kHid * hk::kEmb + hk::kEmb));
    RCHK(grow(ctx, ctx->mlp[6], off));
    char *w = (char *)ctx->mlp[6].p;
    int32_t *score = (int32_t *)(w + o_score);
    float *tgt = (float *)(w + o_tgt);
    RCHK(halign_sw_pairs(ctx, sc, seqs, anc.data(), A, par.data(), score, stream));
    hipLaunchKernelGGL(hk::scale_targets_kernel, dim3((A * 64 + 255) / 256), dim3(256), 0, st, (const int32_t *)score,
                       A * 64, tgt);
    HCHK(hipGetLastError());
    // batch index lists for every step (rows of X_all for a then b, and target slots)
    {
        std::vector<int32_t> order(P), hidx((size_t)nsteps * 2 * B), htix((size_t)nsteps * B);
        for (int q = 0; q < P; ++q) order[q] = q;
        std::vector<int32_t> aord(A);
        for (int q = 0; q < A; ++q) aord[q] = q;
        for (int e = 0; e < opts->epochs; ++e) {
            if (grouped) {   // shuffled anchors, each with its partners in order
                for (int q = A - 1; q > 0; --q) std::swap(aord[q], aord[(int)(splitmix(rs) % (uint64_t)(q + 1))]);
                for (int q = 0; q < P; ++q) order[q] = aord[q / PA] * PA + q % PA;
            } else {
                for (int q = P - 1; q > 0; --q) std::swap(order[q], order[(int)(splitmix(rs) % (uint64_t)(q + 1))]);
            }
            for (int s = 0; s < steps_per_epoch; ++s) {
                const int step = e * steps_per_epoch + s;
                for (int r = 0; r < B; ++r) {
                    const int q = order[s * B + r];
                    const int slot = (q / PA) * 64 + q % PA;
                    hidx[(size_t)step * 2 * B + r] = anc[q / PA];
                    hidx[(size_t)step * 2 * B + B + r] = par[slot];
                    htix[(size_t)step * B + r] = slot;
                }
            }
        }
        HCHK(hipMemcpyAsync(w + o_idx, hidx.data(), 4 * hidx.size(), hipMemcpyHostToDevice, st));
        HCHK(hipMemcpyAsync(w + o_tix, htix.data(), 4 * htix.size(), hipMemcpyHostToDevice, st));
        HCHK(hipStreamSynchronize(st));   // host vectors go out of scope
    }
    uint16_t *X = (uint16_t *)(w + o_X);
    RCHK(halign_featurize(seqs, nullptr, N, X, stream));
    const int64_t nW1 = (int64_t)hk::kFeat * hk::kHid, nW2 = (int64_t)hk::kHid * hk::kEmb;
    float *g = (float *)(w + o_g), *mo = (float *)(w + o_m), *vo = (float *)(w + o_v);
    const int64_t ntot = nW1 + hk::kHid + nW2 + hk::kEmb;
    RCHK(launch_fill((uint32_t *)mo, 0u, ntot, st));
    RCHK(launch_fill((uint32_t *)vo, 0u, ntot, st));
    float *gW1 = g, *gb1 = g + nW1, *gW2 = gb1 + hk::kHid, *gb2 = gW2 + nW2;
    float *mW1 = mo, *mb1 = mo + nW1, *mW2 = mb1 + hk::kHid, *mb2 = mW2 + nW2;
    float *vW1 = vo, *vb1 = vo + nW1, *vW2 = vb1 + hk::kHid, *vb2 = vW2 + nW2;
    uint16_t *Xb = (uint16_t *)(w + o_Xb), *Hb = (uint16_t *)(w + o_Hb);
    float *Z = (float *)(w + o_Z), *E = (float *)(w + o_E), *dE = (float *)(w + o_dE), *tb = (float *)(w + o_tb);
    float *loss = (float *)(w + o_loss);
    halign_model md{pr->W1b, pr->b1, pr->W2b, pr->b2};
    // parameter average (starts from the initial parameters)
    const bool use_ema = opts->ema > 0.f && opts->ema < 1.f;
    float *ema = (float *)(w + o_e);
    float *eW1 = ema, *eb1 = ema + nW1, *eW2 = eb1 + hk::kHid, *eb2 = eW2 + nW2;
    if (use_ema) {
        HCHK(hipMemcpyAsync(eW1, pr->W1, 4 * (size_t)nW1, hipMemcpyDeviceToDevice, st));
        HCHK(hipMemcpyAsync(eb1, pr->b1, 4 * (size_t)hk::kHid, hipMemcpyDeviceToDevice, st));
        HCHK(hipMemcpyAsync(eW2, pr->W2, 4 * (size_t)nW2, hipMemcpyDeviceToDevice, st));
        HCHK(hipMemcpyAsync(eb2, pr->b2, 4 * (size_t)hk::kEmb, hipMemcpyDeviceToDevice, st));
    }
    auto ema_step = [&](const float *p, float *e, int64_t n) -> int {
        hipLaunchKernelGGL(hk::ema_kernel, dim3(grid_for(n, 256, 2048)), dim3(256), 0, st, p, e, n, opts->ema);
        HCHK(hipGetLastError());
        return HALIGN_OK;
    };
    for (int step = 0; step < nsteps; ++step) {
        const int32_t *ix = (const int32_t *)(w + o_idx) + (size_t)step * 2 * B;
        const int32_t *tx = (const int32_t *)(w + o_tix) + (size_t)step * B;
        hipLaunchKernelGGL(hk::gather_rows_kernel, dim3(2 * B), dim3(256), 0, st, (const uint16_t *)X, ix, 2 * B,
                           hk::kFeat, Xb);
        hipLaunchKernelGGL(hk::gather_f32_kernel, dim3((B + 255) / 256), dim3(256), 0, st, (const float *)tgt, tx, B, tb);
        HCHK(hipGetLastError());
        RCHK(halign_mlp_forward(ctx, &md, Xb, 2 * B, Z, Hb, E, stream));
        RCHK(halign_pair_loss_grouped(ctx, E, tb, B, grouped ? PA : 0, opts->group_weight, dE, loss + step, stream));
        RCHK(halign_mlp_backward(ctx, &md, Xb, 2 * B, Z, Hb, dE, gW1, gb1, gW2, gb2, stream));
        const float lr = opts->lr;
        RCHK(halign_adam_step(pr->W1, gW1, mW1, vW1, pr->W1b, nW1, lr, 0.9f, 0.999f, 1e-8f, step + 1, stream));
        RCHK(halign_adam_step(pr->b1, gb1, mb1, vb1, nullptr, hk::kHid, lr, 0.9f, 0.999f, 1e-8f, step + 1, stream));
        RCHK(halign_adam_step(pr->W2, gW2, mW2, vW2, pr->W2b, nW2, lr, 0.9f, 0.999f, 1e-8f, step + 1, stream));
        RCHK(halign_adam_step(pr->b2, gb2, mb2, vb2, nullptr, hk::kEmb, lr, 0.9f, 0.999f, 1e-8f, step + 1, stream));
        if (use_ema) {
            RCHK(ema_step(pr->W1, eW1, nW1));
            RCHK(ema_step(pr->b1, eb1, hk::kHid));
            RCHK(ema_step(pr->W2, eW2, nW2));
            RCHK(ema_step(pr->b2, eb2, hk::kEmb));
        }
    }
    if (use_ema) {   // the averaged parameters become the model
        HCHK(hipMemcpyAsync(pr->W1, eW1, 4 * (size_t)nW1, hipMemcpyDeviceToDevice, st));
        HCHK(hipMemcpyAsync(pr->b1, eb1, 4 * (size_t)hk::kHid, hipMemcpyDeviceToDevice, st));
        HCHK(hipMemcpyAsync(pr->W2, eW2, 4 * (size_t)nW2, hipMemcpyDeviceToDevice, st));
        HCHK(hipMemcpyAsync(pr->b2, eb2, 4 * (size_t)hk::kEmb, hipMemcpyDeviceToDevice, st));
        hipLaunchKernelGGL(hk::f32_to_bf16_kernel, dim3(grid_for(nW1, 256, 2048)), dim3(256), 0, st,
                           (const float *)pr->W1, pr->W1b, nW1);
        hipLaunchKernelGGL(hk::f32_to_bf16_kernel, dim3(grid_for(nW2, 256, 2048)), dim3(256), 0, st,
                           (const float *)pr->W2, pr->W2b, nW2);
        HCHK(hipGetLastError());
    }
    if (loss_host) {
        std::vector<float> hl(nsteps);
        HCHK(hipMemcpyAsync(hl.data(), loss, 4 * (size_t)nsteps, hipMemcpyDeviceToHost, st));
        HCHK(hipStreamSynchronize(st));
        for (int e = 0; e < opts->epochs; ++e) {
            double s = 0;
            for (int q = 0; q < steps_per_epoch; ++q) s += hl[(size_t)e * steps_per_epoch + q];
            loss_host[e] = (float)(s / std::max(1, steps_per_epoch));
        }
    }
    return HALIGN_OK;
}

int halign_center_learned(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs, const halign_model *model,
                          int32_t k, int32_t *cand_host, int32_t *center_host, void *stream) {
    if (!ctx || !center_host || k <= 0) return fail(HALIGN_E_INVALID, "bad arguments");
    RCHK(check_scoring(sc));
    RCHK(check_seqs(seqs));
    RCHK(check_model(model));
    const int N = seqs->n;
    if (N <= 0) return fail(HALIGN_E_INVALID, "empty set");
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    const int kk = std::min<int>(k, N);
    const int CH = 16384;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t r = off; off = (off + bytes + 255) & ~size_t(255); return r; };
    const size_t o_E = take(4 * (size_t)N * hk::kEmb), o_X = take(2 * (size_t)CH * hk::kFeat),
                 o_Hb = take(2 * (size_t)CH * hk::kHid), o_rows = take(4 * (size_t)N), o_u = take(4 * (size_t)N),
                 o_top = take(4 * (size_t)kk), o_sums = take(8 * (size_t)kk);
    RCHK(grow(ctx, ctx->mlp[7], off));
    char *w = (char *)ctx->mlp[7].p;
    float *E = (float *)(w + o_E);
    uint16_t *X = (uint16_t *)(w + o_X), *Hb = (uint16_t *)(w + o_Hb);
    int32_t *rows = (int32_t *)(w + o_rows);
    hipLaunchKernelGGL(hk::iota_kernel, dim3((N + 255) / 256), dim3(256), 0, st, rows, N);
    HCHK(hipGetLastError());
    for (int r0 = 0; r0 < N; r0 += CH) {
        const int nr = std::min(CH, N - r0);
        RCHK(halign_featurize(seqs, rows + r0, nr, X, stream));
        RCHK(halign_mlp_forward(ctx, model, X, nr, nullptr, Hb, E + (size_t)r0 * hk::kEmb, stream));
    }
    int32_t *top = (int32_t *)(w + o_top);
    const int kp = std::min(std::min(ctx->prejudge_cand, 256), N);
    const int np = std::min(ctx->prejudge_part, N);
    if (kp > kk && np > 0) {
        // pre-judge: the top kp by u, scored against a common sample of np
        // partners (evenly spaced indices); the kk best of that sample go on
        RCHK(grow(ctx, ctx->mlp[8], 12 * (size_t)kp + 512));
        int32_t *wide = (int32_t *)ctx->mlp[8].p;
        int64_t *wsum = (int64_t *)((char *)ctx->mlp[8].p + ((4 * (size_t)kp + 255) & ~size_t(255)));
        RCHK(halign_topk_center(ctx, E, N, kp, (float *)(w + o_u), wide, stream));
        std::vector<int32_t> part(np), hw(kp), order(kp);
        for (int q = 0; q < np; ++q) part[q] = (int32_t)((int64_t)q * N / np);
        RCHK(halign_center_judge_sample(ctx, sc, seqs, wide, kp, part.data(), np, wsum, nullptr, stream));
        std::vector<int64_t> hs(kp);
        HCHK(hipMemcpyAsync(hw.data(), wide, 4 * (size_t)kp, hipMemcpyDeviceToHost, st));
        HCHK(hipMemcpyAsync(hs.data(), wsum, 8 * (size_t)kp, hipMemcpyDeviceToHost, st));
        HCHK(hipStreamSynchronize(st));
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
            return hs[x] > hs[y] || (hs[x] == hs[y] && hw[x] < hw[y]);
        });
        std::vector<int32_t> sel(kk);
        for (int q = 0; q < kk; ++q) sel[q] = hw[order[q]];
        HCHK(hipMemcpyAsync(top, sel.data(), 4 * (size_t)kk, hipMemcpyHostToDevice, st));
        HCHK(hipStreamSynchronize(st));
    } else {
        RCHK(halign_topk_center(ctx, E, N, kk, (float *)(w + o_u), top, stream));
    }
    int32_t c = -1;
    RCHK(halign_center_judge(ctx, sc, seqs, top, kk, (int64_t *)(w + o_sums), &c, stream));
    if (cand_host) {
        HCHK(hipMemcpyAsync(cand_host, top, 4 * (size_t)kk, hipMemcpyDeviceToHost, st));
        HCHK(hipStreamSynchronize(st));
    }
    *center_host = c;
    return HALIGN_OK;
}

}  // extern "C"

// ===========================================================================
// Nucleotide center star (trie section)
// ===========================================================================
namespace {

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

// halign_nuc_align; with own_row the center's row is the gapped center itself.
// after: enqueued behind the stretches (each time, where the scratch had to grow
// and they ran again).
static int nuc_align(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs, int32_t center, int32_t k,
                     int32_t *score, uint16_t *ins, uint32_t *aligned, int32_t *G, bool own_row,
                     const std::function<int()> &after, void *stream) {
    if (!ctx || !score || !ins || !aligned) return fail(HALIGN_E_INVALID, "bad arguments");
    RCHK(check_scoring(sc));
    RCHK(check_seqs(seqs));
    if (sc->alphabet < 5) return fail(HALIGN_E_UNSUPPORTED, "nucleotide alphabet needs codes 0..4 (A C G T other)");
    if (k < 1 || k > 32) return fail(HALIGN_E_UNSUPPORTED, "segment length %d outside 1..32", k);
    const int N = seqs->n;
    if (center < 0 || center >= N) return fail(HALIGN_E_INVALID, "center %d of %d", center, N);
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    const int64_t *oh = seqs->offsets_host;
    const int m = (int)(oh[center + 1] - oh[center]);
    const uint8_t *dc = seqs->residues + oh[center];
    Scoring S;
    hk::PrepArgs pa{};
    RCHK(upload_matrix(ctx, sc, st, &S, &pa));
    // the center's segments: at most this many different strings, so the table
    // is at most half full
    const int nsg = m / k;
    const int distinct = k < 12 ? std::min(nsg, 1 << (2 * k)) : nsg;
    int lg_t = 6;
    while ((1 << lg_t) < 2 * distinct) ++lg_t;
    const int T = 1 << lg_t;
    // scan chunks: sequence x covers the match starts 0 .. n - k in chunks
    int64_t nchunk = 0;
    int longest = 0;
    for (int x = 0; x < N; ++x) {
        const int64_t n = oh[x + 1] - oh[x], w = std::max<int64_t>(0, n - k + 1);
        nchunk += (w + hk::kNucChunk - 1) / hk::kNucChunk;
        longest = std::max<int>(longest, (int)n);
    }
    // device tables: segment table and its making, chunk bases, counters; per
    // chunk its count; a place per residue for the matches
    const size_t o_tk = 0, o_ts = al256(8 * (size_t)T), o_sk = o_ts + al256(4 * (size_t)T),
                 o_ss = o_sk + al256(8 * (size_t)nsg + 8), o_st = o_ss + al256(4 * (size_t)nsg + 4),
                 o_cb = o_st + al256(4 * (size_t)nsg + 4), o_n = o_cb + al256(8 * (size_t)(N + 1)),
                 o_cc = o_n + 8 * hk::kNucCounts, o_cm = o_cc + al256(4 * (size_t)nchunk + 4),
                 tab_bytes = o_cm + 4 * (size_t)oh[N] + 4;
    RCHK(grow(ctx, ctx->nuctab, tab_bytes));
    char *tb = (char *)ctx->nuctab.p;
    const int aw = (m + 31) / 32;
    {   // the code check, and the vectors (ins as words plus an odd tail), G and the counters zeroed
        const int64_t n16 = (int64_t)N * (m + 1);
        pa.z[0] = (uint32_t *)ins;
        pa.nz[0] = n16 / 2;
        pa.z[1] = aligned;
        pa.nz[1] = (int64_t)N * aw;
        pa.z[2] = (uint32_t *)G;
        pa.nz[2] = G ? m + 1 : 0;
        pa.z[3] = (uint32_t *)(tb + o_n);
        pa.nz[3] = 2 * hk::kNucCounts;
        pa.tail16 = (n16 & 1) ? ins + (n16 - 1) : nullptr;
        RCHK(validate_codes(ctx, sc->alphabet, seqs->residues, oh[N], nullptr, 0, st, pa));
    }
    hk::NucSetup su{};
    su.center = dc;
    su.m = m;
    su.k = k;
    su.nsg = nsg;
    su.alpha = S.alpha;
    su.lg_t = lg_t;
    su.mat = S.dmat;
    su.tkey = (unsigned long long *)(tb + o_tk);
    su.tseg = (int32_t *)(tb + o_ts);
    su.segkey = (unsigned long long *)(tb + o_sk);
    su.segscore = (int32_t *)(tb + o_ss);
    su.segstate = (int32_t *)(tb + o_st);
    su.off = seqs->offsets;
    su.nseq = N;
    su.cbase = (int64_t *)(tb + o_cb);
    hipLaunchKernelGGL(hk::nuc_setup_kernel, dim3(2), dim3(1024), 0, st, su);
    HCHK(hipGetLastError());
    hk::NucArgs a{};
    a.res = seqs->residues;
    a.off = seqs->offsets;
    a.nseq = N;
    a.center = dc;
    a.m = m;
    a.k = k;
    a.tkey = su.tkey;
    a.tseg = su.tseg;
    a.lg_t = lg_t;
    a.segscore = su.segscore;
    a.mat = S.dmat;
    a.alpha = S.alpha;
    a.go = S.goe - S.ge;
    a.ge = S.ge;
    a.cbase = su.cbase;
    a.nchunk = nchunk;
    a.ccount = (int32_t *)(tb + o_cc);
    a.cmatch = (uint32_t *)(tb + o_cm);
    a.score = score;
    a.ins = ins;
    a.aligned = aligned;
    a.aw = aw;
    a.G = G;
    a.gskip = center;
    a.own_row = own_row ? 1 : 0;
    a.count = (unsigned long long *)(tb + o_n);
    a.lane_min = hk::kNucLaneMin;
    if (const char *e = getenv("HALIGN_NUC_LANES")) a.lane_min = atoll(e);   // test knob: lanes from this many narrow stretches
    if (nchunk > 0) {
        if (k <= hk::kNucWaveMaxK) {
            // 16 wavefronts per workgroup share the table, two workgroups a CU
            const int64_t waves = (int64_t)ctx->num_cu * 2 * 16, longest = (nchunk + N - 1) / N;
            a.wparts = (int)std::max<int64_t>(1, std::min(waves / N, longest));
            const int64_t items = (int64_t)N * a.wparts;
            const unsigned grid = (unsigned)std::min<int64_t>((items + 15) / 16, (int64_t)ctx->num_cu * 2);
            if (k <= hk::kNucKey32) hipLaunchKernelGGL(hk::nuc_scan_wave_kernel<uint32_t>, dim3(grid), dim3(1024), 0, st, a);
            else hipLaunchKernelGGL(hk::nuc_scan_wave_kernel<unsigned long long>, dim3(grid), dim3(1024), 0, st, a);
        } else {
            hipLaunchKernelGGL(hk::nuc_scan_kernel, dim3((unsigned)((nchunk + 255) / 256)), dim3(256), 0, st, a);
        }
        HCHK(hipGetLastError());
    }
    // LDS of the chain for a quarter more matches than anchors can fit (each
    // position of the center matches once in a related sequence), so that several
    // workgroups share a CU (1,035 anchors: 18 KB).  A sequence with more, as short
    // segments match by chance, is chained by one lane in global arrays.  Up to two
    // sequences per CU, which fit with the largest LDS too, there is LDS for half more
    // than the chance matches (of `indexed` strings that occur once in the center,
    // among 4^k), and for kChainLdsMax where that fell short in every eighth sequence (an uneven
    // composition), here and in later calls of this k and number of segments.
    // Whole calls with matches in global arrays against LDS, sequences of 16,500: 100 with
    // k = 7 4.55 against 3.71 ms, with k = 9 and 80% A and T 3.32 against 2.76; 672, which then
    // no longer fit at once, 5.15 against 7.13 and 3.72 against 5.22.
    const int fit = std::min(longest, m) / k;
    int cap = std::min(hk::kChainLdsMax, (fit + fit / 4 + 127) & ~63);
    const bool roomy = N <= 2 * ctx->num_cu && cap < hk::kChainLdsMax;
    if (roomy) {
        const double strings = std::pow(4.0, k), indexed = nsg * std::exp(-nsg / strings);
        const double chance = std::min<double>(hk::kChainLdsMax, 1.5 * longest * indexed / strings);
        cap = std::min(hk::kChainLdsMax, (fit + fit / 4 + (int)chance + 127) & ~63);
        if (ctx->nuc_crowded[0] == k && ctx->nuc_crowded[1] == nsg) cap = hk::kChainLdsMax;
    }
    // The lists and the scratch of the stretches are as large as the last calls
    // needed, or a first guess: the kernels count what they need, and where it
    // is more the buffers grow and the stretches run again, the chain too where it
    // had no place for a match or a stretch.
    // The guess: eight stretches a sequence (672 genomes of 16,569 bases: seven), fewer
    // where sequences are short, four million at most (1.6 GB in all).
    int64_t list = std::max<int64_t>(ctx->nuc_list, std::min({(int64_t)N * 8, oh[N] / 32, (int64_t)1 << 22}) + 4096);
    int64_t codes = std::max<int64_t>(ctx->nuc_codes, list * 64), rows = std::max<int64_t>(ctx->nuc_rows, list * 8);
    int64_t big = ctx->nuc_big;
    for (bool chain = true;;) {
        const size_t lc = (size_t)list;
        const size_t l_nd = 0, l_wd = al256(16 * lc), l_no = l_wd + al256(16 * lc), l_wo = l_no + al256(16 * lc),
                     l_nx = l_wo + al256(16 * lc), l_wx = l_nx + al256(4 * lc), l_big = l_wx + al256(4 * lc),
                     scr_bytes = l_big + 20 * (size_t)big + 4;
        RCHK(grow(ctx, ctx->nucscr, scr_bytes));
        const size_t d_co = al256(8 * (size_t)rows);
        RCHK(grow(ctx, ctx->nucdp, d_co + 4 * (size_t)codes));
        ctx->nuc_list = list;   // (kept once they are allocated)
        ctx->nuc_codes = codes;
        ctx->nuc_rows = rows;
        ctx->nuc_big = big;
        char *sb = (char *)ctx->nucscr.p;
        a.nd = (int4 *)(sb + l_nd);
        a.wd = (int4 *)(sb + l_wd);
        a.no = (longlong2 *)(sb + l_no);
        a.wo = (longlong2 *)(sb + l_wo);
        a.nx = (int32_t *)(sb + l_nx);
        a.wx = (int32_t *)(sb + l_wx);
        a.big = (int32_t *)(sb + l_big);
        a.bigcap = big;
        a.listcap = list;
        a.rows = (int2 *)ctx->nucdp.p;
        a.codes = (uint32_t *)((char *)ctx->nucdp.p + d_co);
        a.rowcap = rows;
        a.codecap = codes;
        a.flag = (const uint32_t *)ctx->counter.p + 8;
        a.mail = ctx->mail_dev;
        a.seq = ctx->mail_dev ? ++ctx->mail_seq : 0;
        a.chain_cap = cap;
        if (chain) {
            hipLaunchKernelGGL(hk::nuc_chain_kernel, dim3((unsigned)N), dim3(256), hk::nuc_chain_lds_bytes(cap, aw), st, a);
            HCHK(hipGetLastError());
        }
        // (33 KB of LDS: four workgroups a CU)
        const int64_t sgrid = std::max<int64_t>(1, std::min<int64_t>(((int64_t)N * 8 + 3) / 4, (int64_t)ctx->num_cu * 4));
        hipLaunchKernelGGL(hk::nuc_stretch_kernel, dim3((unsigned)sgrid), dim3(256), 0, st, a);
        HCHK(hipGetLastError());
        RCHK(after());
        if (!chain) break;   // (its counts were read the first time)
        int64_t need[5];   // boundary entries, code words, narrow (front | back << 32), wide, big
        if (ctx->mail_dev) {
            RCHK(mail_wait(ctx, a.seq, st));
            for (int c = 0; c < 5; ++c) need[c] = ctx->mail_host[3 + c];
            *ctx->flag_host = (int)ctx->mail_host[2];
        } else {
            RCHK(flag_fetch(ctx, st));
            HCHK(hipMemcpy2DAsync(need, 8, a.count, 256, 8, 5, hipMemcpyDeviceToHost, st));
            HCHK(hipStreamSynchronize(st));
        }
        ctx->stage_pending = false;
        const bool crowded = roomy && cap < hk::kChainLdsMax && need[4] > (int64_t)N * cap / 8;
        if (crowded) {
            ctx->nuc_crowded[0] = k;
            ctx->nuc_crowded[1] = nsg;
        }
        const int64_t narrow = (need[2] & 0xffffffffll) + (int64_t)((uint64_t)need[2] >> 32);
        chain = narrow > a.listcap || need[3] > a.listcap || need[4] > a.bigcap;
        if (!chain && need[0] <= a.rowcap && need[1] <= a.codecap) break;
        RCHK(validate_check(ctx));
        if (narrow >= ((int64_t)1 << 31) || need[3] >= ((int64_t)1 << 31))
            return fail(HALIGN_E_UNSUPPORTED, "%lld stretches", (long long)(narrow + need[3]));
        rows = std::max(rows, need[0]);
        codes = std::max(codes, need[1]);
        list = std::max({list, narrow, need[3]});
        if (crowded) cap = hk::kChainLdsMax;
        big = std::max(big, need[4]);
        if (chain) RCHK(launch_fill((uint32_t *)a.count, 0u, 2 * hk::kNucCounts, st));
    }
    return validate_check(ctx);
}

extern "C" {

int halign_nuc_align(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs, int32_t center, int32_t k,
                     int32_t *score, uint16_t *ins, uint32_t *aligned, int32_t *G, void *stream) {
    return nuc_align(ctx, sc, seqs, center, k, score, ins, aligned, G, false, [] { return HALIGN_OK; }, stream);
}

int halign_nuc_msa(halign_ctx *ctx, const halign_scoring *sc, const halign_seqs *seqs, int32_t center, int32_t k,
                   int32_t *score, halign_alloc_fn alloc, void *user, uint8_t **msa, int64_t *width_host,
                   void *stream) {
    if (!ctx || !alloc || !msa || !width_host || !score) return fail(HALIGN_E_INVALID, "bad arguments");
    int longest = 0;
    RCHK(check_seqs(seqs, &longest));
    const int N = seqs->n;
    if (center < 0 || center >= N) return fail(HALIGN_E_INVALID, "center %d of %d", center, N);
    hipStream_t st = (hipStream_t)stream;
    const int m = (int)(seqs->offsets_host[center + 1] - seqs->offsets_host[center]);
    const int aw = (m + 31) / 32;
    // vectors, G, col in the ctx's MSA scratch
    const size_t o_ins = 0, o_al = (2 * (size_t)N * (m + 1) + 255) & ~(size_t)255,
                 o_g = o_al + ((4 * (size_t)N * aw + 255) & ~(size_t)255), o_col = o_g + ((4 * (size_t)(m + 1) + 255) & ~(size_t)255),
                 bytes = o_col + 8 * (size_t)(m + 1);
    RCHK(grow(ctx, ctx->msabuf, bytes));
    char *mb = (char *)ctx->msabuf.p;
    uint16_t *ins = (uint16_t *)(mb + o_ins);
    uint32_t *al = (uint32_t *)(mb + o_al);
    int32_t *G = (int32_t *)(mb + o_g);
    int64_t *col = (int64_t *)(mb + o_col);
    int64_t width = 0;
    RCHK(nuc_align(ctx, sc, seqs, center, k, score, ins, al, G, true,
                   [&] { return merge_offsets(ctx, G, m + 1, col, &width, st); }, stream));
    uint8_t *out = (uint8_t *)alloc((size_t)N * (size_t)width, user);
    if (!out && width > 0) return fail(HALIGN_E_NOMEM, "allocator returned NULL for %lld bytes", (long long)(N * width));
    RCHK(emit_rows(ctx, seqs, m, ins, al, G, col, width, out, longest, st));
    *msa = out;
    *width_host = width;
    return HALIGN_OK;
}

}  // extern "C"

// ===========================================================================
// Phylogeny (NJ section, Fig. 4): p-distances, neighbour joining, the sampled
// clustering and the merged tree
// ===========================================================================
namespace {

inline size_t al256z(size_t b) { return (b + 255) & ~(size_t)255; }

// The distance launch: whole width per tile, or, when the tiles are too few to
// fill the chip, column slices and a pass that adds them.
int pdist_launch(halign_ctx *ctx, hk::PdArgs a, int64_t tiles, hipStream_t st) {
    // below 2,048 tiles (eight workgroups per CU, what its registers hold) as
    // many slices, of at least 256 columns, as bring the workgroups to 2,048 or
    // past it (under 4,095: 134 MB of counts): 3,001 x 4,030 rows, 2,256 workgroups,
    // 0.62 ms (0.68 unsliced, 0.68 up to 1,024 workgroups), 672 x 18,611 0.20 (1.07,
    // 0.23), 64 x 18,000 0.05 (0.85, 0.05)
    int64_t nslice = tiles < 2048 ? std::min<int64_t>((a.width + 255) / 256, (2047 + tiles) / tiles) : 1;
    nslice = std::max<int64_t>(1, nslice);
    a.cslice = std::max<int64_t>(1, ((a.width + nslice - 1) / nslice + hk::kPdChunk - 1) / hk::kPdChunk) * hk::kPdChunk;
    nslice = std::max<int64_t>(1, (a.width + a.cslice - 1) / a.cslice);
    a.nslice = (int)nslice;
    a.acc = nullptr;
    if (nslice > 1) {
        RCHK(grow(ctx, ctx->njacc, (size_t)(tiles * nslice) * 16 * 256 * sizeof(int2)));
        a.acc = (int2 *)ctx->njacc.p;
    }
    hipLaunchKernelGGL(hk::pdist_kernel, dim3((unsigned)(tiles * nslice)), dim3(256), 0, st, a);
    HCHK(hipGetLastError());
    if (nslice > 1) {
        hipLaunchKernelGGL(hk::pd_final_kernel, dim3((unsigned)(tiles * 16)), dim3(256), 0, st, a);
        HCHK(hipGetLastError());
    }
    return HALIGN_OK;
}

// Upload rows and the group table, then one pdist launch over every group's
// tiles.  Synchronises the stream after the upload (the host vectors may go).
int pdist_groups(halign_ctx *ctx, const uint8_t *msa, int64_t width, const std::vector<int32_t> &rows,
                 std::vector<hk::PdGroup> &groups, double *D, int32_t *mism, int32_t *comp, hipStream_t st) {
    int64_t tiles = 0;
    for (auto &g : groups) {
        g.tiles_b = (g.nb + hk::kPdTile - 1) / hk::kPdTile;
        g.tile0 = tiles;
        tiles += hk::pd_tiles(g);
    }
    if (tiles == 0) return HALIGN_OK;
    if (tiles > 0x7fffffff) return fail(HALIGN_E_UNSUPPORTED, "%lld distance tiles", (long long)tiles);
    const size_t o_g = al256z(4 * rows.size());
    RCHK(grow(ctx, ctx->njrows, o_g + sizeof(hk::PdGroup) * groups.size()));
    char *b = (char *)ctx->njrows.p;
    if (!rows.empty()) HCHK(hipMemcpyAsync(b, rows.data(), 4 * rows.size(), hipMemcpyHostToDevice, st));
    HCHK(hipMemcpyAsync(b + o_g, groups.data(), sizeof(hk::PdGroup) * groups.size(), hipMemcpyHostToDevice, st));
    hk::PdArgs a{};
    a.msa = msa; a.width = width; a.rows_a = a.rows_b = (const int32_t *)b;
    a.groups = (const hk::PdGroup *)(b + o_g); a.ngroups = (int)groups.size();
    a.D = D; a.mism = mism; a.comp = comp;
    RCHK(pdist_launch(ctx, a, tiles, st));
    HCHK(hipStreamSynchronize(st));
    return HALIGN_OK;
}

// Neighbour joining over groups (each D at its d0 in dbase, modified); the
// trees come back to the host: tree g at t0 = 2 * (sum of earlier n) + g.
// The one-workgroup joins of several problems (each group's offsets filled
// in), enqueued on st; nj_groups_finish copies the trees to the host.
struct NjLaunch {
    size_t o_p = 0, o_b = 0, o_nd = 0;
    int64_t nt = 0;
    size_t G = 0;
};

int nj_groups_launch(halign_ctx *ctx, std::vector<hk::NjGroup> &groups, double *dbase, NjLaunch &L, hipStream_t st) {
    int64_t ns = 0, nt = 0;
    int nmax = 0;
    for (auto &g : groups) {
        g.s0 = ns;
        g.t0 = nt;
        ns += g.n;
        nt += 2 * (int64_t)g.n + 1;
        nmax = std::max(nmax, g.n);
    }
    const size_t G = groups.size();
    const size_t o_r = 0, o_id = al256z(8 * ns), o_p = o_id + al256z(4 * ns), o_b = o_p + al256z(4 * nt),
                 o_nd = o_b + al256z(8 * nt), o_g = o_nd + al256z(4 * G), o_act = o_g + al256z(sizeof(hk::NjGroup) * G),
                 bytes = o_act + al256z(ns);
    RCHK(grow(ctx, ctx->njS, bytes));
    char *b = (char *)ctx->njS.p;
    HCHK(hipMemcpyAsync(b + o_g, groups.data(), sizeof(hk::NjGroup) * G, hipMemcpyHostToDevice, st));
    hk::NjArgs a{(const hk::NjGroup *)(b + o_g), dbase, (double *)(b + o_r), (uint8_t *)(b + o_act),
                 (int32_t *)(b + o_id), (int32_t *)(b + o_p), (double *)(b + o_b), (int32_t *)(b + o_nd)};
    const int bs = nmax > 128 ? 1024 : 256;
    const size_t lds = hk::nj_lds_bytes(nmax);   // at most 55 KiB
    hipLaunchKernelGGL(hk::nj_kernel, dim3((unsigned)G), dim3(bs), lds, st, a, lds > 0 ? 1 : 0);
    HCHK(hipGetLastError());
    L.o_p = o_p;
    L.o_b = o_b;
    L.o_nd = o_nd;
    L.nt = nt;
    L.G = G;
    return HALIGN_OK;
}

int nj_groups_finish(halign_ctx *ctx, const NjLaunch &L, std::vector<int32_t> &parent, std::vector<double> &blen,
                     std::vector<int32_t> &nodes, hipStream_t st) {
    // parents, lengths and node counts lie together: one copy
    const size_t bytes = L.o_nd + 4 * L.G - L.o_p;
    RCHK(grow_host(ctx->njout, bytes));
    const char *h = (const char *)ctx->njout.p;
    HCHK(hipMemcpyAsync(ctx->njout.p, (const char *)ctx->njS.p + L.o_p, bytes, hipMemcpyDeviceToHost, st));
    HCHK(hipStreamSynchronize(st));
    parent.assign((const int32_t *)h, (const int32_t *)h + L.nt);
    blen.assign((const double *)(h + L.o_b - L.o_p), (const double *)(h + L.o_b - L.o_p) + L.nt);
    nodes.assign((const int32_t *)(h + L.o_nd - L.o_p), (const int32_t *)(h + L.o_nd - L.o_p) + L.G);
    return HALIGN_OK;
}

int nj_groups(halign_ctx *ctx, std::vector<hk::NjGroup> &groups, double *dbase, std::vector<int32_t> &parent,
              std::vector<double> &blen, std::vector<int32_t> &nodes, hipStream_t st) {
    NjLaunch L;
    RCHK(nj_groups_launch(ctx, groups, dbase, L, st));
    return nj_groups_finish(ctx, L, parent, blen, nodes, st);
}

// Problems above this many nodes are joined over the whole chip; smaller ones
// of a tree one workgroup each, all in one launch.
constexpr int kNjBigMin = 256;
// Problems from this many nodes that are joined alone (halign_nj, the seeds of a
// tree) go to the mesh too: 10 nodes 135 us against 161 on one workgroup, 64
// 385 against 840, 256 1,520 against 3,740 (whole calls).
constexpr int kNjMeshMin = 8;

// Whether a problem of n nodes fits the mesh of workgroups that hold 16 rows each in LDS.
bool nj_mesh_ok(const halign_ctx *ctx, int n) {
    const char *env = getenv("HALIGN_NJ_MESH");   // test knob: 0 = the other kernels
    return n <= hk::kNjMeshMax && (n + hk::kNjMeshRows - 1) / hk::kNjMeshRows <= ctx->num_cu &&
           hk::nj_mesh_lds(n) + 1024 <= ctx->lds_max && !(env && atoi(env) == 0);
}

// Scratch of one problem that is joined alone.  Parents, lengths and the node
// count lie together: they come back in one copy.
struct NjAlone {
    size_t o_p, o_b, o_nodes, o_fail, o_mesh, o_M;
    int G;   // workgroups of the mesh
    hk::NjBigArgs a;
};
int nj_alone(halign_ctx *ctx, double *D, int n, bool mesh, NjAlone *w) {
    const int64_t nn = (int64_t)n * n;
    const int nparts = (int)std::max<int64_t>(1, std::min<int64_t>(2048, (nn + 255) / 256));
    const size_t nt = 2 * (size_t)n + 1;
    w->G = (n + hk::kNjMeshRows - 1) / hk::kNjMeshRows;
    const size_t o_r = 0, o_id = al256z(8 * (size_t)n);
    w->o_p = o_id + al256z(4 * (size_t)n);
    w->o_b = w->o_p + al256z(4 * nt);
    w->o_nodes = w->o_b + al256z(8 * nt);
    w->o_fail = w->o_nodes + 64;
    const size_t o_part = w->o_nodes + 256, o_pd = o_part + al256z(sizeof(hk::NjBest) * nparts),
                 o_ctrl = o_pd + al256z(8 * (size_t)nparts), o_act = o_ctrl + 256;
    w->o_mesh = o_act + al256z(n);
    w->o_M = w->o_mesh + (mesh ? al256z(8 * (3 * (size_t)n + 9 * (size_t)w->G)) : 0);
    RCHK(grow(ctx, ctx->njB, w->o_M + (mesh ? al256z(8 * (size_t)nn) : 0)));
    RCHK(grow_host(ctx->njout, w->o_nodes + 4 - w->o_p));
    char *b = (char *)ctx->njB.p;
    w->a = hk::NjBigArgs{n, D, (double *)(b + o_r), (uint8_t *)(b + o_act), (int32_t *)(b + o_id), (int32_t *)(b + w->o_p),
                         (double *)(b + w->o_b), (hk::NjBest *)(b + o_part), (double *)(b + o_pd), nparts,
                         (hk::NjCtrl *)(b + o_ctrl)};
    return HALIGN_OK;
}

// The last joins on the matrix M, and the tree to the host (2n + 1 entries; -1
// nodes where *failed is set).
int nj_alone_finish(halign_ctx *ctx, const NjAlone &w, double *M, const uint32_t *failed, std::vector<int32_t> &parent,
                    std::vector<double> &blen, int *nodes, hipStream_t st) {
    char *b = (char *)ctx->njB.p;
    const size_t nt = 2 * (size_t)w.a.n + 1;
    hk::NjBigArgs f = w.a;
    f.D = M;
    hipLaunchKernelGGL(hk::nj_big_finish_kernel, dim3(1), dim3(1), 0, st, f, failed, (int32_t *)(b + w.o_nodes));
    HCHK(hipGetLastError());
    const char *h = (const char *)ctx->njout.p;
    HCHK(hipMemcpyAsync(ctx->njout.p, b + w.o_p, w.o_nodes + 4 - w.o_p, hipMemcpyDeviceToHost, st));
    HCHK(hipStreamSynchronize(st));
    parent.assign((const int32_t *)h, (const int32_t *)h + nt);
    blen.assign((const double *)(h + w.o_b - w.o_p), (const double *)(h + w.o_b - w.o_p) + nt);
    int32_t nd = 0;
    memcpy(&nd, h + w.o_nodes - w.o_p, 4);
    *nodes = nd;
    return HALIGN_OK;
}

// Neighbour joining of one problem on the mesh: D (device, n x n, not modified);
// the tree to the host (2n + 1 entries).  *nodes < 0: the mesh left the problem
// to the other kernels (its workgroups were not resident together, or a sum of
// distances is infinite or NaN, whose order among pairs is the other kernels').
int nj_mesh(halign_ctx *ctx, double *D, int n, std::vector<int32_t> &parent, std::vector<double> &blen, int *nodes,
            hipStream_t st) {
    NjAlone w;
    RCHK(nj_alone(ctx, D, n, true, &w));
    char *b = (char *)ctx->njB.p;
    hk::NjMeshArgs g{n, w.G, D, (double *)(b + w.o_M), (uint64_t *)(b + w.o_mesh), (uint64_t *)(b + w.o_mesh) + 3 * (size_t)n,
                     (uint32_t *)(b + w.o_fail), hk::kNjSpin, w.a};
    if (const char *e = getenv("HALIGN_NJ_SPIN")) g.spin = atoi(e);   // test knob: 0 = every wait gives up at once
    RCHK(launch_fill((uint32_t *)(b + w.o_mesh), 0xffffffffu, 2 * (3 * (int64_t)n + 9 * (int64_t)w.G), st));
    RCHK(launch_fill(g.failed, 0u, 1, st));
    hipLaunchKernelGGL(hk::nj_mesh_kernel, dim3((unsigned)w.G), dim3(256), hk::nj_mesh_lds(n), st, g);
    HCHK(hipGetLastError());
    return nj_alone_finish(ctx, w, g.M, g.failed, parent, blen, nodes, st);
}

// The same over the whole chip, three launches a join; D is modified.
int nj_big(halign_ctx *ctx, double *D, int n, std::vector<int32_t> &parent, std::vector<double> &blen, int *nodes,
           hipStream_t st) {
    NjAlone w;
    RCHK(nj_alone(ctx, D, n, false, &w));
    const hk::NjBigArgs &a = w.a;
    const unsigned rg = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(hk::nj_big_init_kernel, dim3(rg), dim3(256), 0, st, a);
    HCHK(hipGetLastError());
    for (int t = 0; t < n - 3; ++t) {
        hipLaunchKernelGGL(hk::nj_big_rows_kernel, dim3((unsigned)((n + hk::kNjRowsCols - 1) / hk::kNjRowsCols)),
                           dim3(256), 0, st, a);
        hipLaunchKernelGGL(hk::nj_big_q_kernel, dim3((unsigned)a.nparts), dim3(256), 0, st, a);
        hipLaunchKernelGGL(hk::nj_big_join_kernel, dim3(1), dim3(256), 0, st, a);
    }
    HCHK(hipGetLastError());
    return nj_alone_finish(ctx, w, D, nullptr, parent, blen, nodes, st);
}

// One problem of a tree by itself: on the mesh where it fits, else over the chip.
int nj_one(halign_ctx *ctx, double *D, int n, std::vector<int32_t> &parent, std::vector<double> &blen, int *nodes,
           hipStream_t st) {
    if (nj_mesh_ok(ctx, n)) {
        RCHK(nj_mesh(ctx, D, n, parent, blen, nodes, st));
        if (*nodes >= 0) return HALIGN_OK;
    }
    return nj_big(ctx, D, n, parent, blen, nodes, st);
}

// labels[i] = nearest of the nb columns of D (na x nb, device), to the host
// labels[g][i] = nearest of the nb columns of group g's block (D + o, na x
// nb): every group's launch, then one copy to the host
int nearest_groups(halign_ctx *ctx, const double *D, const std::vector<hk::PdGroup> &gr,
                   std::vector<std::vector<int32_t>> &label, hipStream_t st) {
    size_t tot = 0;
    for (auto &g : gr) tot += (size_t)std::max(0, g.na);
    RCHK(grow(ctx, ctx->njS, al256z(4 * tot + 4)));
    int32_t *lab = (int32_t *)ctx->njS.p;
    size_t at = 0;
    for (auto &g : gr) {
        if (g.na > 0 && g.nb > 0)
            hipLaunchKernelGGL(hk::nearest_kernel, dim3((unsigned)((g.na + 255) / 256)), dim3(256), 0, st, D + g.o,
                               (int64_t)g.nb, g.na, g.nb, lab + at);
        at += (size_t)std::max(0, g.na);
    }
    HCHK(hipGetLastError());
    std::vector<int32_t> all(tot);
    if (tot > 0) HCHK(hipMemcpyAsync(all.data(), lab, 4 * tot, hipMemcpyDeviceToHost, st));
    HCHK(hipStreamSynchronize(st));
    label.resize(gr.size());
    at = 0;
    for (size_t gi = 0; gi < gr.size(); ++gi) {
        const int na = std::max(0, gr[gi].na);
        label[gi].assign(all.begin() + at, all.begin() + at + na);
        at += na;
    }
    return HALIGN_OK;
}

int nearest_host(halign_ctx *ctx, const double *D, int na, int nb, std::vector<int32_t> &label, hipStream_t st) {
    RCHK(grow(ctx, ctx->njS, al256z(4 * (size_t)na)));
    int32_t *lab = (int32_t *)ctx->njS.p;
    hipLaunchKernelGGL(hk::nearest_kernel, dim3((unsigned)((na + 255) / 256)), dim3(256), 0, st, D, (int64_t)nb, na,
                       nb, lab);
    HCHK(hipGetLastError());
    label.resize(na);
    HCHK(hipMemcpyAsync(label.data(), lab, 4 * (size_t)na, hipMemcpyDeviceToHost, st));
    HCHK(hipStreamSynchronize(st));
    return HALIGN_OK;
}

}  // namespace

extern "C" {

int halign_pdist(halign_ctx *ctx, const uint8_t *msa, int32_t n, int64_t width, const int32_t *a_rows, int32_t na,
                 const int32_t *b_rows, int32_t nb, double *D, int32_t *mism, int32_t *comp, void *stream) {
    if (!ctx || n < 0 || width < 0 || na < 0 || nb < 0 || ((int64_t)na * nb > 0 && (!D || (!msa && width > 0))))
        return fail(HALIGN_E_INVALID, "bad arguments");
    if ((!a_rows && na > n) || (!b_rows && nb > n)) return fail(HALIGN_E_INVALID, "row count above n");
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    if ((int64_t)na * nb == 0) return HALIGN_OK;
    hk::PdArgs a{};
    a.msa = msa; a.width = width; a.rows_a = a_rows; a.rows_b = b_rows;
    a.D = D; a.mism = mism; a.comp = comp;
    a.g.na = na; a.g.nb = nb; a.g.ld = nb;
    a.g.tiles_b = (nb + hk::kPdTile - 1) / hk::kPdTile;
    a.g.sym = a_rows == b_rows && na == nb;   // the same rows on both sides: one triangle is computed
    if ((int64_t)((na + hk::kPdTile - 1) / hk::kPdTile) * a.g.tiles_b > 0x7fffffff)
        return fail(HALIGN_E_UNSUPPORTED, "distance tiles");
    return pdist_launch(ctx, a, hk::pd_tiles(a.g), st);
}

int halign_nj(halign_ctx *ctx, const double *D, int32_t n, int32_t *parent_host, double *blen_host, int32_t *nodes,
              void *stream) {
    if (!ctx || n < 1 || !D || !parent_host || !blen_host || !nodes) return fail(HALIGN_E_INVALID, "bad arguments");
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    const size_t bytes = 8 * (size_t)n * n;
    RCHK(grow(ctx, ctx->njD, bytes));
    HCHK(hipMemcpyAsync(ctx->njD.p, D, bytes, hipMemcpyDeviceToDevice, st));
    std::vector<int32_t> parent, nd;
    std::vector<double> blen;
    int nn = -1;
    if (n >= kNjMeshMin && nj_mesh_ok(ctx, n)) RCHK(nj_mesh(ctx, (double *)ctx->njD.p, n, parent, blen, &nn, st));
    if (nn < 0 && n > kNjBigMin) RCHK(nj_big(ctx, (double *)ctx->njD.p, n, parent, blen, &nn, st));
    if (nn >= 0) {
        nd.assign(1, nn);
    } else {
        std::vector<hk::NjGroup> groups(1);
        groups[0].n = n;
        groups[0].d0 = 0;
        RCHK(nj_groups(ctx, groups, (double *)ctx->njD.p, parent, blen, nd, st));
    }
    memcpy(parent_host, parent.data(), 4 * (size_t)nd[0]);
    memcpy(blen_host, blen.data(), 8 * (size_t)nd[0]);
    *nodes = nd[0];
    return HALIGN_OK;
}

int halign_nj_tree(halign_ctx *ctx, const uint8_t *msa, int32_t n, int64_t width, const int32_t *perm_host,
                   int32_t *parent_host, double *blen_host, int32_t *nodes, void *stream) {
    if (!ctx || n < 1 || width < 0 || (!msa && width > 0) || !perm_host || !parent_host || !blen_host || !nodes)
        return fail(HALIGN_E_INVALID, "bad arguments");
    {   // a permutation of 0 .. n-1
        std::vector<char> seen(n, 0);
        for (int t = 0; t < n; ++t) {
            const int v = perm_host[t];
            if (v < 0 || v >= n || seen[v]) return fail(HALIGN_E_INVALID, "perm is not a permutation of 0..%d", n - 1);
            seen[v] = 1;
        }
    }
    HCHK(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    const int N = n, S = (N + 9) / 10;
    std::vector<int32_t> seed(perm_host, perm_host + S);
    // Where all rows' distances are cheap (up to 2e10 pair-columns in one
    // triangle, about 0.5 ms) and few (768 rows, 4.7 MB), they are computed at once
    // and copied to the host, which labels and divides from them: a divide pass
    // costs a distance launch, a nearest launch and two waits otherwise, about
    // 0.2 ms, and there are up to 20.  The host's part grows with the square of the
    // rows: of 300 to 18,000 columns, a launch per step takes 4.0 times as long at
    // 64 rows, 1.58 at 400, 1.15 at 672, 1.04 at 760, 0.99 at 840, 0.96 at 1,000,
    // 0.71 at 2,000 (whole trees, geometric means).
    // The values are the same either way.
    const char *env_full = getenv("HALIGN_NJ_FULL");   // test knob: 0 = per step
    const bool full =
        N <= 768 && 0.5 * (double)N * N * (double)width <= 2e10 && !(env_full && atoi(env_full) == 0);
    const double *F = nullptr;
    // the first of `nb` rows b with the smallest distance to row x
    auto nearest = [&](int x, const int32_t *rb, int nb) {
        const double *f = F + (size_t)x * N;
        int best = 0;
        double bd = f[rb[0]];
        for (int e = 1; e < nb; ++e)
            if (f[rb[e]] < bd) {
                bd = f[rb[e]];
                best = e;
            }
        return best;
    };
    // every row against the sample: nearest seed
    std::vector<int32_t> label;
    if (full) {
        const size_t bytes = 8 * (size_t)N * N;
        RCHK(grow(ctx, ctx->njF, bytes));
        RCHK(grow_host(ctx->njhost, bytes));
        hk::PdArgs a{};
        a.msa = msa; a.width = width; a.D = (double *)ctx->njF.p;
        a.g.na = a.g.nb = N; a.g.ld = N; a.g.sym = 1;
        a.g.tiles_b = (N + hk::kPdTile - 1) / hk::kPdTile;
        RCHK(pdist_launch(ctx, a, hk::pd_tiles(a.g), st));
        HCHK(hipMemcpyAsync(ctx->njhost.p, ctx->njF.p, bytes, hipMemcpyDeviceToHost, st));
        HCHK(hipStreamSynchronize(st));
        F = (const double *)ctx->njhost.p;
        label.resize(N);
        for (int x = 0; x < N; ++x) label[x] = nearest(x, seed.data(), S);
    } else {
        std::vector<int32_t> rows(N + S);
        for (int x = 0; x < N; ++x) rows[x] = x;
        for (int c = 0; c < S; ++c) rows[N + c] = seed[c];
        std::vector<hk::PdGroup> gr(1);
        gr[0] = hk::PdGroup{0, N, N, S, 0, S, 0, 0, 0, 0};
        RCHK(grow(ctx, ctx->njD, 8 * (size_t)N * S));
        RCHK(pdist_groups(ctx, msa, width, rows, gr, (double *)ctx->njD.p, nullptr, nullptr, st));
        RCHK(nearest_host(ctx, (const double *)ctx->njD.p, N, S, label, st));
    }
    int K = S;
    std::vector<int> size(N + 1, 0);
    for (int x = 0; x < N; ++x) size[label[x]]++;
    if (ctx->progress) fprintf(stderr, "halign_nj_tree: %d rows labelled against %d seeds\n", N, S);
    // clusters of fewer than 3 rows join the cluster of the nearest seed
    bool small = false;
    for (int c = 0; c < K; ++c) small = small || (size[c] > 0 && size[c] < 3);
    if (small && K > 1) {
        std::vector<int> to(K);   // cluster a small one moved to (itself when kept)
        for (int c = 0; c < K; ++c) to[c] = c;
        // the seeds' distances on the host
        std::vector<double> dss((size_t)S * S);
        if (full) {
            for (int c = 0; c < S; ++c)
                for (int e = 0; e < S; ++e) dss[(size_t)c * S + e] = F[(size_t)seed[c] * N + seed[e]];
        } else {
            std::vector<int32_t> rows(seed.begin(), seed.begin() + S);
            std::vector<hk::PdGroup> gr(1);
            gr[0] = hk::PdGroup{0, 0, S, S, 0, S, 0, 0, 0, 1};
            RCHK(grow(ctx, ctx->njD, 8 * (size_t)S * S));
            RCHK(pdist_groups(ctx, msa, width, rows, gr, (double *)ctx->njD.p, nullptr, nullptr, st));
            HCHK(hipMemcpyAsync(dss.data(), ctx->njD.p, 8 * (size_t)S * S, hipMemcpyDeviceToHost, st));
            HCHK(hipStreamSynchronize(st));
        }
        for (int c = 0; c < K; ++c) {
            if (size[c] == 0 || size[c] >= 3) continue;
            const double *drow = dss.data() + (size_t)c * S;
            double best = 0.0;
            int bc = -1;
            for (int e = 0; e < K; ++e) {
                if (e == c || size[e] == 0) continue;
                if (bc < 0 || drow[e] < best) {
                    best = drow[e];
                    bc = e;
                }
            }
            if (bc < 0) continue;
            to[c] = bc;   // the rows follow at the end, along the chain of moves
            size[bc] += size[c];
            size[c] = 0;
        }
        for (int x = 0; x < N; ++x) {
            int c = label[x];
            while (to[c] != c) c = to[c];
            label[x] = c;
        }
    }
    {   // renumber the clusters left, in order
        std::vector<int> map(K);
        int K2 = 0;
        for (int c = 0; c < K; ++c) map[c] = size[c] > 0 ? K2++ : -1;
        for (int c = 0; c < K; ++c)
            if (map[c] >= 0) {
                seed[map[c]] = seed[c];
                size[map[c]] = size[c];
            }
        for (int x = 0; x < N; ++x) label[x] = map[label[x]];
        K = K2;
    }
    // clusters of more than ceil(N / 10) rows are divided until none is left:
    // among their first ceil(size / 10) rows in permutation order (nearest),
    // or in runs of ceil(N / 10) rows in permutation order when one seed
    // takes them all; empty clusters are dropped after each pass
    for (;;) {
        bool big = false;
        for (int c = 0; c < K; ++c) big = big || size[c] > S;
        if (!big) break;
        std::vector<int32_t> nseed, nlab(N);
        // the big clusters' rows and new seeds, one distance group each
        std::vector<int32_t> rows;
        std::vector<hk::PdGroup> gr;
        std::vector<int> gbase;                     // per group: its cluster's first new seed
        std::vector<std::vector<int32_t>> mem(K);
        for (int x = 0; x < N; ++x)
            if (size[label[x]] > S) mem[label[x]].push_back(x);
        int64_t dtot = 0;
        std::vector<int32_t> kpos(K, -1);   // a kept cluster's seed position in nseed
        for (int c = 0; c < K; ++c) {
            if (size[c] <= S) {
                kpos[c] = (int32_t)nseed.size();
                nseed.push_back(seed[c]);
                continue;
            }
            const int nsd = (size[c] + 9) / 10;
            const int base = (int)nseed.size();
            for (int t = 0; t < N && (int)nseed.size() - base < nsd; ++t)
                if (label[perm_host[t]] == c) nseed.push_back(perm_host[t]);
            const int64_t r0 = (int64_t)rows.size();
            rows.insert(rows.end(), mem[c].begin(), mem[c].end());
            rows.insert(rows.end(), nseed.begin() + base, nseed.end());
            const int nm = (int)mem[c].size();
            gr.push_back(hk::PdGroup{r0, r0 + nm, nm, nsd, dtot, nsd, 0, 0, 0, 0});
            gbase.push_back(base);
            dtot += (int64_t)nm * nsd;
        }
        for (int x = 0; x < N; ++x)   // rows of kept clusters: their seed's position
            if (kpos[label[x]] >= 0) nlab[x] = kpos[label[x]];
        // the nearest new seed of every row of each divided cluster
        std::vector<std::vector<int32_t>> glab(gr.size());
        if (full) {
            for (size_t q = 0; q < gr.size(); ++q) {
                glab[q].resize(gr[q].na);
                for (int t = 0; t < gr[q].na; ++t)
                    glab[q][t] = nearest(rows[gr[q].a0 + t], rows.data() + gr[q].b0, gr[q].nb);
            }
        } else {   // on the GPU (one launch per cluster, one copy back)
            RCHK(grow(ctx, ctx->njD, 8 * (size_t)dtot));
            RCHK(pdist_groups(ctx, msa, width, rows, gr, (double *)ctx->njD.p, nullptr, nullptr, st));
            RCHK(nearest_groups(ctx, (const double *)ctx->njD.p, gr, glab, st));
        }
        // nearest new seed per row (ties to the earlier), or runs in permutation order
        std::vector<int> remap(nseed.size(), -1);
        {
            // rebuild nseed in order, replacing each divided cluster's seeds by
            // runs where needed
            size_t gi = 0;
            std::vector<int32_t> res;
            int at = 0;   // position in nseed
            for (int c = 0; c < K; ++c) {
                if (size[c] <= S) {
                    remap[at] = (int)res.size();
                    res.push_back(nseed[at]);
                    ++at;
                    continue;
                }
                const hk::PdGroup &g = gr[gi];
                const int nm = g.na, nsd = g.nb, base = gbase[gi];
                const std::vector<int32_t> &lab = glab[gi];
                bool split = false;
                for (int t = 1; t < nm; ++t) split = split || lab[t] != lab[0];
                if (split) {
                    const int r0 = (int)res.size();
                    for (int e = 0; e < nsd; ++e) res.push_back(nseed[base + e]);
                    for (int t = 0; t < nm; ++t) nlab[mem[c][t]] = r0 + lab[t];
                } else {
                    int cnt = 0;
                    for (int t = 0; t < N; ++t) {
                        const int x = perm_host[t];
                        if (label[x] != c) continue;
                        if (cnt % S == 0) res.push_back(x);
                        nlab[x] = (int32_t)res.size() - 1;
                        ++cnt;
                    }
                }
                at += nsd;
                ++gi;
            }
            // the kept clusters' labels were set against nseed positions: move them
            for (int x = 0; x < N; ++x)
                if (size[label[x]] <= S) nlab[x] = remap[nlab[x]];
            nseed.swap(res);
        }
        // drop empty clusters, keeping the order
        const int NK = (int)nseed.size();
        std::vector<int> sz(NK, 0), map(NK);
        for (int x = 0; x < N; ++x) sz[nlab[x]]++;
        int K2 = 0;
        for (int c = 0; c < NK; ++c) map[c] = sz[c] > 0 ? K2++ : -1;
        seed.assign(K2, 0);
        size.assign(std::max(N + 1, K2), 0);
        for (int c = 0; c < NK; ++c)
            if (map[c] >= 0) {
                seed[map[c]] = nseed[c];
                size[map[c]] = sz[c];
            }
        for (int x = 0; x < N; ++x) label[x] = map[nlab[x]];
        K = K2;
        if (ctx->progress) fprintf(stderr, "halign_nj_tree: divide pass, %d clusters\n", K);
    }
    // distance matrices: each cluster over its rows (row order), then the seeds
    std::vector<int32_t> rows;
    std::vector<int64_t> coff(K + 1, 0);
    std::vector<int> csize(K, 0);
    for (int x = 0; x < N; ++x) csize[label[x]]++;
    for (int c = 0; c < K; ++c) coff[c + 1] = coff[c] + csize[c];
    rows.resize(N + K);
    {
        std::vector<int64_t> at(coff.begin(), coff.end() - 1);
        for (int x = 0; x < N; ++x) rows[at[label[x]]++] = x;
        for (int c = 0; c < K; ++c) rows[N + c] = seed[c];
    }
    if (ctx->progress) {
        int mx = 0;
        for (int c = 0; c < K; ++c) mx = std::max(mx, csize[c]);
        fprintf(stderr, "halign_nj_tree: %d rows, %d clusters (largest %d rows), %d seeds joined last\n", N, K, mx, K);
    }
    std::vector<hk::PdGroup> gr(K + 1);
    std::vector<hk::NjGroup> ng(K + 1);
    int64_t dtot = 0;
    for (int c = 0; c <= K; ++c) {
        const int64_t r0 = c < K ? coff[c] : N;
        const int sz = c < K ? csize[c] : K;
        gr[c] = hk::PdGroup{r0, r0, sz, sz, dtot, sz, 1, 0, 0, 1};
        ng[c].n = sz;
        ng[c].d0 = dtot;
        dtot += (int64_t)sz * sz;
    }
    if (full) {   // every matrix out of the full one
        const size_t nr = rows.size(), o_lx = al256z(4 * nr), o_ls = o_lx + al256z(4 * nr),
                     bytes = o_ls + sizeof(hk::PdList) * (size_t)(K + 1);
        RCHK(grow(ctx, ctx->njD, 8 * (size_t)dtot));
        RCHK(grow(ctx, ctx->njrows, bytes));
        RCHK(stage_begin(ctx));
        char *hs = nullptr;
        RCHK(stage_host(ctx, bytes, &hs));
        memcpy(hs, rows.data(), 4 * nr);
        int32_t *lx = (int32_t *)(hs + o_lx);
        hk::PdList *ls = (hk::PdList *)(hs + o_ls);
        for (int c = 0; c <= K; ++c) {
            ls[c] = hk::PdList{gr[c].a0, ng[c].d0, ng[c].n};
            for (int t = 0; t < ng[c].n; ++t) lx[gr[c].a0 + t] = c;
        }
        char *d = (char *)ctx->njrows.p;
        HCHK(hipMemcpyAsync(d, hs, bytes, hipMemcpyHostToDevice, st));
        stage_copied(ctx);
        RCHK(stage_close(ctx, st));
        hipLaunchKernelGGL(hk::pd_gather_kernel, dim3((unsigned)nr), dim3(256), 0, st, (const double *)ctx->njF.p, N,
                           (const int32_t *)d, (const int32_t *)(d + o_lx), (const hk::PdList *)(d + o_ls),
                           (double *)ctx->njD.p);
        HCHK(hipGetLastError());
    } else {
        // clusters of at most 64 rows, consecutive in `rows`, share 64-row tiles:
        // one square group over the span (its pairs across clusters are computed
        // and not used), each cluster's block then copied to its own matrix; a
        // distance depends on its two rows alone, so the values are the same
        std::vector<hk::PdGroup> gp;
        std::vector<hk::PdExtract> ext;
        int64_t ttot = dtot;
        for (int c = 0; c < K;) {
            if (csize[c] > hk::kPdTile) {
                gp.push_back(gr[c++]);
                continue;
            }
            const int first = c;
            const int64_t R0 = coff[c];
            int span = 0;
            while (c < K && csize[c] <= hk::kPdTile && span + csize[c] <= hk::kPdTile) span += csize[c++];
            if (c - first == 1) {
                gp.push_back(gr[first]);
                continue;
            }
            gp.push_back(hk::PdGroup{R0, R0, span, span, ttot, span, 1, 0, 0, 1});
            for (int q = first; q < c; ++q)
                if (csize[q] > 0) {
                    const int64_t off = coff[q] - R0;
                    ext.push_back(hk::PdExtract{ttot + off * span + off, span, ng[q].d0, csize[q]});
                }
            ttot += (int64_t)span * span;
        }
        gp.push_back(gr[K]);
        RCHK(grow(ctx, ctx->njD, 8 * (size_t)ttot));
        RCHK(pdist_groups(ctx, msa, width, rows, gp, (double *)ctx->njD.p, nullptr, nullptr, st));
        if (!ext.empty()) {
            RCHK(grow(ctx, ctx->njrows, sizeof(hk::PdExtract) * ext.size()));
            HCHK(hipMemcpyAsync(ctx->njrows.p, ext.data(), sizeof(hk::PdExtract) * ext.size(), hipMemcpyHostToDevice,
                                st));
            hipLaunchKernelGGL(hk::pd_extract_kernel, dim3((unsigned)ext.size()), dim3(256), 0, st,
                               (double *)ctx->njD.p, (const hk::PdExtract *)ctx->njrows.p);
            HCHK(hipGetLastError());
            HCHK(hipStreamSynchronize(st));   // the host vector was copied from
        }
    }
    // the joins: small problems in one launch, large ones over the chip; tree
    // g at tp/tb offset ng[g].t0 (2n + 1 entries each), node count tn[g]
    std::vector<int32_t> tp, tn(K + 1);
    std::vector<double> tb;
    {
        // joined by itself: large problems, and the seeds' where the mesh takes it
        auto alone = [&](int c) {
            return ng[c].n > kNjBigMin || (c == K && ng[c].n >= kNjMeshMin && nj_mesh_ok(ctx, ng[c].n));
        };
        std::vector<hk::NjGroup> small;
        std::vector<int> sidx;
        int64_t nt = 0;
        for (int c = 0; c <= K; ++c) {
            ng[c].t0 = nt;
            nt += 2 * (int64_t)ng[c].n + 1;
            if (!alone(c)) {
                small.push_back(ng[c]);
                sidx.push_back(c);
            }
        }
        tp.assign(nt, 0);
        tb.assign(nt, 0.0);
        // the small problems on a second stream, beside the joins of the large
        // (their matrices, scratch and trees are disjoint), once the distances
        // are in place
        bool any_big = false;
        for (int c = 0; c <= K; ++c) any_big = any_big || alone(c);
        hipStream_t sst = st;
        if (any_big && !small.empty()) {
            if (!ctx->aux_stream) HCHK(hipStreamCreateWithFlags(&ctx->aux_stream, hipStreamNonBlocking));
            if (!ctx->ev_nj) HCHK(hipEventCreateWithFlags(&ctx->ev_nj, hipEventDisableTiming));
            sst = ctx->aux_stream;
            HCHK(hipEventRecord(ctx->ev_nj, st));
            HCHK(hipStreamWaitEvent(sst, ctx->ev_nj, 0));
        }
        NjLaunch L;
        if (!small.empty()) RCHK(nj_groups_launch(ctx, small, (double *)ctx->njD.p, L, sst));
        for (int c = 0; c <= K; ++c) {
            if (!alone(c)) continue;
            if (ctx->progress) fprintf(stderr, "halign_nj_tree: joining %d nodes over the chip\n", ng[c].n);
            std::vector<int32_t> bp;
            std::vector<double> bb;
            int nn = 0;
            const int rc = nj_one(ctx, (double *)ctx->njD.p + ng[c].d0, ng[c].n, bp, bb, &nn, st);
            if (rc != HALIGN_OK) {   // the small joins finish before the scratch can be reused
                if (sst != st) (void)hipStreamSynchronize(sst);
                return rc;
            }
            std::copy(bp.begin(), bp.end(), tp.begin() + ng[c].t0);
            std::copy(bb.begin(), bb.end(), tb.begin() + ng[c].t0);
            tn[c] = nn;
        }
        if (!small.empty()) {
            std::vector<int32_t> sp, sn;
            std::vector<double> sb;
            RCHK(nj_groups_finish(ctx, L, sp, sb, sn, sst));
            for (size_t q = 0; q < small.size(); ++q) {
                const int c = sidx[q];
                std::copy(sp.begin() + small[q].t0, sp.begin() + small[q].t0 + 2 * ng[c].n + 1, tp.begin() + ng[c].t0);
                std::copy(sb.begin() + small[q].t0, sb.begin() + small[q].t0 + 2 * ng[c].n + 1, tb.begin() + ng[c].t0);
                tn[c] = sn[q];
            }
        }
        if (ctx->progress) fprintf(stderr, "halign_nj_tree: %zu problems joined in one launch\n", small.size());
    }
    // the merge, node numbering as documented
    int next = N;
    std::vector<int> croot(K);
    for (int c = 0; c < K; ++c) {
        const int nn = tn[c], sz = csize[c];
        const int32_t *lp = tp.data() + ng[c].t0;
        const double *lb = tb.data() + ng[c].t0;
        const int32_t *mem = rows.data() + coff[c];
        for (int v = 0; v < nn; ++v) {
            const int gv = v < sz ? mem[v] : next + v - sz;
            const int pv = lp[v];
            parent_host[gv] = pv < 0 ? -1 : (pv < sz ? mem[pv] : next + pv - sz);
            blen_host[gv] = lb[v];
            if (pv < 0) croot[c] = gv;
        }
        next += nn - sz;
    }
    {
        const int nn = tn[K];
        const int32_t *lp = tp.data() + ng[K].t0;
        const double *lb = tb.data() + ng[K].t0;
        for (int v = 0; v < nn; ++v) {
            const int gv = v < K ? croot[v] : next + v - K;
            const int pv = lp[v];
            parent_host[gv] = pv < 0 ? -1 : (pv < K ? croot[pv] : next + pv - K);
            blen_host[gv] = pv < 0 ? 0.0 : lb[v];
        }
        next += nn - K;
    }
    *nodes = next;
    return HALIGN_OK;
}

}  // extern "C"

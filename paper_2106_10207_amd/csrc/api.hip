// C ABI of libdedloc (declared in include/dedloc.h): argument validation,
// host-side integer work (shard bounds, peer weights, LAMB tile tables) and
// the launch sequence of each call.  All arithmetic on vector data runs in
// the kernels of kernels.hip.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/dedloc.h"
#include "dedloc_internal.h"

using namespace dedloc;

// The workspace of dedloc_round_noalloc.  In host code `scratch` names a
// host-side stand-in, not device memory: its device address (one per GPU)
// comes from hipGetSymbolAddress and only that address is handed to kernels.
static __device__ __align__(256) unsigned char scratch[DEDLOC_NOALLOC_SCRATCH_BYTES];

namespace {

thread_local std::string g_err;

int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

int hip_fail(hipError_t e, const char *what) {
    return fail(DEDLOC_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

bool aligned(const void *p, size_t a) { return ((uintptr_t)p % a) == 0; }

// ------------------------------------------------------------ profiling
enum Kind {
    K_ENCODE_FP16, K_DECODE_FP16, K_ENCODE_I8, K_DECODE_I8, K_REDUCE_FP16, K_REDUCE_I8,
    K_LAMB_A_F32, K_LAMB_A_FP16, K_LAMB_A_I8, K_LAMB_A_FUSED_FP16, K_LAMB_B,
    K_LARS_A_F32, K_LARS_A_FP16, K_LARS_A_I8, K_LARS_A_FUSED_FP16, K_LARS_B,
    K_ACCUMULATE, K_FINALIZE_FP16, K_FINALIZE_I8, K_FILL, K_COUNT
};
const char *const kKindNames[K_COUNT] = {
    "encode_fp16", "decode_fp16", "encode_i8", "decode_i8", "reduce_fp16", "reduce_i8",
    "lamb_a_f32", "lamb_a_fp16", "lamb_a_i8", "lamb_a_fused_fp16", "lamb_b",
    "lars_a_f32", "lars_a_fp16", "lars_a_i8", "lars_a_fused_fp16", "lars_b",
    "accumulate", "finalize_fp16", "finalize_i8", "fill_zero"};

struct Profiler {
    std::mutex mu;
    bool on = false;
    uint32_t cap = 0;
    std::vector<hipEvent_t> ev;     // 2 per recorded launch
    std::vector<int> kind;
    size_t used = 0;
} g_prof;

// Run `launch` (returning hipError_t), bracketed by events when profiling.
template <typename F>
hipError_t timed(int kind, hipStream_t s, F launch) {
    std::unique_lock<std::mutex> lk(g_prof.mu);
    if (!g_prof.on || g_prof.used >= g_prof.cap) {
        lk.unlock();
        return launch();
    }
    const size_t i = g_prof.used++;
    while (g_prof.ev.size() < 2 * g_prof.used) {
        hipEvent_t e;
        hipError_t r = hipEventCreate(&e);
        if (r != hipSuccess) return r;
        g_prof.ev.push_back(e);
    }
    g_prof.kind.resize(g_prof.used);
    g_prof.kind[i] = kind;
    hipError_t r = hipEventRecord(g_prof.ev[2 * i], s);
    if (r != hipSuccess) return r;
    r = launch();
    if (r != hipSuccess) return r;
    return hipEventRecord(g_prof.ev[2 * i + 1], s);
}

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Host copy of dedloc_weights' definition: exact integer total, exactly
// converted, one fp32 division per peer.
int compute_weights(const uint32_t *counts, uint32_t n, float *w) {
    uint64_t W = 0;
    for (uint32_t p = 0; p < n; p++) W += counts[p];
    if (W == 0) return fail(DEDLOC_ERR_ZERO_WEIGHT, "every peer has zero samples");
    if (W > (1u << 24)) return fail(DEDLOC_ERR_INVALID_ARG, "total sample count %llu exceeds 2^24",
                                    (unsigned long long)W);
    for (uint32_t p = 0; p < n; p++) w[p] = (float)counts[p] / (float)W;
    return DEDLOC_OK;
}

int check_codec(int32_t codec, uint32_t block, bool allow_f32) {
    if (codec == DEDLOC_CODEC_FP16) return DEDLOC_OK;
    if (codec == DEDLOC_CODEC_F32 && allow_f32) return DEDLOC_OK;
    if (codec == DEDLOC_CODEC_I8) {
        if (block != DEDLOC_I8_BLOCK)
            return fail(DEDLOC_ERR_INVALID_ARG, "int8 block must be %d (got %u)", DEDLOC_I8_BLOCK, block);
        return DEDLOC_OK;
    }
    return fail(DEDLOC_ERR_INVALID_ARG, "unknown codec %d", codec);
}

static_assert(DEDLOC_MAX_GROUP_SIZE <= kMaxPeers, "a group must fit one launch's peer table");

// Active peers: those with counts > 0, in ascending order, with weights.
struct PeerList {
    std::vector<const void *> codes;
    std::vector<const float *> scales;
    std::vector<float> w;
    std::vector<uint32_t> index;  // the caller's peer index
    uint32_t n() const { return (uint32_t)w.size(); }
};

int build_peers(const void *const *codes, const float *const *scales, const uint32_t *counts,
                uint32_t n, int32_t codec, PeerList &pl, bool check_ptrs = true) {
    if (!codes || !counts) return fail(DEDLOC_ERR_INVALID_ARG, "peer_codes and counts must not be NULL");
    if (n == 0 || n > DEDLOC_MAX_PEERS)
        return fail(DEDLOC_ERR_INVALID_ARG, "n_peers must be in [1, %d] (got %u)", DEDLOC_MAX_PEERS, n);
    if (codec == DEDLOC_CODEC_I8 && !scales)
        return fail(DEDLOC_ERR_INVALID_ARG, "int8 messages need peer_scales");
    std::vector<float> w(n);
    int rc = compute_weights(counts, n, w.data());
    if (rc) return rc;
    pl = PeerList();
    if (!check_ptrs) return DEDLOC_OK;  // nothing will be read at all
    for (uint32_t p = 0; p < n; p++) {
        if (counts[p] == 0) continue;  // weight 0: never read
        if (!codes[p]) return fail(DEDLOC_ERR_INVALID_ARG, "peer %u has samples but a NULL message", p);
        if (!aligned(codes[p], 16)) return fail(DEDLOC_ERR_ALIGN, "peer %u message is not 16-byte aligned", p);
        const float *sc = nullptr;
        if (codec == DEDLOC_CODEC_I8) {
            if (!scales[p]) return fail(DEDLOC_ERR_INVALID_ARG, "peer %u has samples but NULL scales", p);
            if (!aligned(scales[p], 4)) return fail(DEDLOC_ERR_ALIGN, "peer %u scales not 4-byte aligned", p);
            sc = scales[p];
        }
        pl.codes.push_back(codes[p]);
        pl.scales.push_back(sc);
        pl.w.push_back(w[p]);
        pl.index.push_back(p);
    }
    return DEDLOC_OK;
}

// Active peers [lo, hi) as one launch's table (hi - lo <= kMaxPeers).
PeerTable table_of(const PeerList &pl, uint32_t lo, uint32_t hi) {
    PeerTable pt;
    memset(&pt, 0, sizeof pt);
    for (uint32_t p = lo; p < hi; p++) {
        pt.codes[pt.n] = pl.codes[p];
        pt.scales[pt.n] = pl.scales[p];
        pt.w[pt.n] = pl.w[p];
        pt.n++;
    }
    return pt;
}

// A plain reduce: every peer of the table in one group writing `out`.
GroupTable single_group(const PeerTable &pt, void *out, float *out_scales) {
    GroupTable gt;
    memset(&gt, 0, sizeof gt);
    gt.pt = pt;
    gt.gbegin[0] = 0;
    gt.gbegin[1] = pt.n;
    gt.out[0] = out;
    gt.out_scales[0] = out_scales;
    gt.n_groups = 1;
    return gt;
}

// More active peers than one launch's table holds need the fp32 mean buffer
// to carry the running sum between launches.
int check_chain(const PeerList &pl, const float *mean) {
    if (pl.n() > (uint32_t)kMaxPeers && !mean)
        return fail(DEDLOC_ERR_INVALID_ARG, "%u peers with samples (more than %d) need out_mean", pl.n(), kMaxPeers);
    return DEDLOC_OK;
}

// Start of the last launch's peers when peers [0, n) are reduced in
// launches of kMaxPeers.
uint32_t last_batch(uint32_t n) { return n == 0 ? 0 : (n - 1) / kMaxPeers * kMaxPeers; }

// The local peer as seen by a launch of active peers [a, b): its position
// relative to a, or -1 if the launch does not hold it.
LocalArgs local_in(const LocalArgs &la, uint32_t a, uint32_t b) {
    LocalArgs r = la;
    r.pos = (la.pos >= 0 && (uint32_t)la.pos >= a && (uint32_t)la.pos < b) ? la.pos - (int32_t)a : -1;
    return r;
}

// Compute units of the current device (256 if it cannot be asked).
uint32_t cu_count() {
    static std::atomic<int> known[64];
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    n = known[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        known[dev].store(n, std::memory_order_relaxed);
    }
    return (uint32_t)n;
}

// Reduce peers [lo, hi) of the list in launches of kMaxPeers, chained through
// `mean`; the launch holding peer hi - 1 encodes into out / out_scales when
// `encode` is set.  Peers before lo must already be summed into `mean`.
// la.pos: the local peer's position in the list (-1: none; fp16 only).
int run_reduce(int32_t codec, const PeerList &pl, uint32_t lo, uint32_t hi, bool encode, uint64_t len,
               void *out, float *out_scales, float *mean, const LocalArgs &la, hipStream_t s) {
    for (uint32_t a = lo; a < hi; a += kMaxPeers) {
        const uint32_t b = std::min(hi, a + (uint32_t)kMaxPeers);
        const GroupTable gt = single_group(table_of(pl, a, b), out, out_scales);
        const ChainArgs ca = {a > 0 ? mean : nullptr, mean, encode && b == hi, local_in(la, a, b), 1, 0, 0};
        const hipError_t e = codec == DEDLOC_CODEC_FP16
                                 ? timed(K_REDUCE_FP16, s, [&] { return launch_reduce_fp16(gt, len, ca, s); })
                                 : timed(K_REDUCE_I8, s, [&] { return launch_reduce_i8(gt, len, ca, cu_count(), s); });
        if (e != hipSuccess) return hip_fail(e, "reduce launch");
    }
    return DEDLOC_OK;
}

// Work table of an optimizer: tensors in launch chunks of at most
// kChunkTensors.
struct Plan {
    std::vector<Chunk> chunks;
    bool one_pass = false;  // LAMB in one pass (else the two passes)
    bool nt = false;        // LARS: non-temporal accesses to the state
    size_t ws_part = 0, ws_trust = 0, ws_total = 0;
};

int check_tensors(uint64_t P, const uint64_t *off, uint32_t T) {
    if (!off) return fail(DEDLOC_ERR_INVALID_ARG, "offsets must not be NULL");
    if (T == 0) return fail(DEDLOC_ERR_INVALID_ARG, "n_tensors must be >= 1");
    if (off[0] != 0 || off[T] != P)
        return fail(DEDLOC_ERR_INVALID_ARG, "tensor offsets must start at 0 and end at P");
    for (uint32_t t = 0; t < T; t++) {
        if (off[t + 1] < off[t]) return fail(DEDLOC_ERR_INVALID_ARG, "tensor offsets decrease at %u", t);
        if (off[t] % kVec) return fail(DEDLOC_ERR_ALIGN, "tensor offset %u is not a multiple of 8", t);
        if (off[t + 1] - off[t] >= (1ull << 32))
            return fail(DEDLOC_ERR_INVALID_ARG, "tensor %u has 2^32 or more elements", t);
    }
    return DEDLOC_OK;
}

// LAMB's one pass (x and u held on chip until the tensor's ratio is known)
// moves 28 instead of 40 bytes of state per element, but its persistent grid
// and the wait for every tensor's ratio cost more than that saves on small
// vectors and on tables of many small tensors.  Measured, one pass against
// two, steps: 2M elements in 20 tensors 21.0 / 19.2 us, 4M in one 28.7 / 30.6, 8M
// in 20 49.9 / 55.7, 4M in 200 52 / 41, 17.7M in 25 98 / 123.  Rounds: 9M in 5
// (int8) 88.0 / 98.6, 9M in 300 138 / 122, 9M in 12 80.8 / 78.6, 12M in one 99.9 /
// 98.9, 17M in 12 140.6 / 144.8, 20M in 30 162 / 171, 2^30 in 1024 8.9 / 10.1 ms.
// The mean size is a coarse line.  ResNet-50's 161 tensors (159k elements on
// average, 107 of them of at most 2048) lie below it: 32 peers 452 / 442 us on the
// same buffers and 472 / 464 after a cache flush, but with three sets of buffers
// in turn 466 / 494, 16 peers 310 / 334, int8 254 / 278.
constexpr uint64_t kOnePassElements = 1ull << 23;       // a message or fp32 gradient
constexpr uint64_t kOnePassElementsPeers = 1ull << 24;  // the fused average
constexpr uint64_t kOnePassPerTensor = 1ull << 18;
// Of a tensor the grid's line holds its last 2 * 768 units on 256 CUs, 6.3M
// elements; the rest takes a second pass all the same, and the fused average is
// then slower in the persistent grid than in two plain passes.  So it takes the
// one pass where the line holds a third of the elements.  One pass against two,
// on the same buffers, 2, 8, 16 and 60 peers, us: tensors of 12M elements (held
// 52%) 457 / 475, 574 / 596, 739 / 780, 1078 / 1075; 16.8M (37%) 394 / 397, 493 /
// 498, 627 / 659, 1021 / 1009; 33M (19%) 277 / 268, 346 / 338, 430 / 441, 1028 /
// 1010.  Three sets of buffers in turn, 33M, 4, 8, 16, 32, 41 and 60 peers: 304 /
// 286, 321 / 316, 449 / 439, 615 / 624, 734 / 740, 971 / 975.  A message or fp32
// gradient gains throughout (one tensor of 33M 223 / 235, of 2^30 7.8 / 8.2 ms).
// LARS: x and v of 2^24 elements are 128 MB, half of the Infinity Cache.
// Non-temporal accesses beyond: 8.5M and 9M elements 61.6 / 65.0 and 75.2 / 78.0
// us, 12M equal, 18M 148.6 / 141.8, 26M 201.5 / 198.1, 40M 232.5 / 222.5
// (without / with).
constexpr uint64_t kNtElements = 1ull << 24;

// Units of a tensor that a persistent grid on this many CUs holds: a unit leaves
// the line kLineUnits turns after it entered, and the last unit of its tensor
// must have been taken a turn before that.
uint32_t held_units(uint32_t cus) { return (kLineUnits - 1) * cus * kLineGroups; }

void make_plan(int opt, bool peers, uint64_t P, const uint64_t *off, const uint8_t *flags, uint32_t T, Plan &pl) {
    uint64_t full = 0;  // tensors with elements
    for (uint32_t t = 0; t < T; t++) full += off[t + 1] > off[t];
    pl.one_pass = opt == kOptLamb && P >= (peers ? kOnePassElementsPeers : kOnePassElements) && P / full >= kOnePassPerTensor;
    if (pl.one_pass && peers) {
        const uint64_t line = (uint64_t)held_units(cu_count()) * 2 * kRow;
        uint64_t held = 0;
        for (uint32_t t = 0; t < T; t++) held += std::min(off[t + 1] - off[t], line);
        pl.one_pass = 3 * held >= P;
    }
    pl.nt = P >= kNtElements;
    const uint32_t per = pl.one_pass ? 2 : 1;  // rows per work item
    pl.chunks.clear();
    uint32_t all_rows = 0;
    uint32_t t0 = 0;
    while (t0 < T) {
        Chunk c;
        memset(&c, 0, sizeof c);
        c.base = off[t0];
        c.t0 = t0;
        c.row_base = all_rows;
        uint32_t items = 0, odd = 0, k = 0;
        // take tensors while they fit the table and the chunk spans < 2^32 elements
        while (k < (uint32_t)kChunkTensors && t0 + k < T && off[t0 + k + 1] - c.base < (1ull << 32)) {
            c.start[k] = (uint32_t)(off[t0 + k] - c.base);
            c.begin[k] = items;
            c.odd_before[k] = (uint8_t)odd;
            c.flags[k] = flags ? flags[t0 + k] : 0;
            const uint32_t rows = (uint32_t)((off[t0 + k + 1] - off[t0 + k] + kRow - 1) / kRow);
            items += (rows + per - 1) / per;
            odd += rows % 2;
            all_rows += rows;
            k++;
        }
        if (k == 0) k = 1;  // unreachable: every tensor was checked to span < 2^32 elements
        c.nt = k;
        c.start[k] = (uint32_t)(off[t0 + k] - c.base);
        c.begin[k] = items;
        pl.chunks.push_back(c);
        t0 += k;
    }
    pl.ws_part = round_up((size_t)all_rows * 2 * sizeof(double), 256);
    pl.ws_trust = round_up((size_t)T * sizeof(unsigned long long), 256);
    pl.ws_total = 256 + pl.ws_part + pl.ws_trust;
}

// The counter comes first: calls with different tables that take turns on
// one workspace all advance the same one.
LineWs carve_line(const Plan &pl, void *ws) {
    char *b = (char *)ws;
    return {(uint32_t *)b, (unsigned long long *)(b + 128), (unsigned long long *)(b + 256),
            (unsigned long long *)(b + 256 + pl.ws_part)};
}

TileWs carve_tiles(const Plan &pl, void *ws) {
    char *b = (char *)ws;
    return {(double *)(b + 256), (unsigned long long *)(b + 256 + pl.ws_part), (uint32_t *)b};
}

// Polls of a tensor's published trust ratio in pass B before a workgroup
// computes it itself (dedloc_test_trust_polls).
std::atomic<uint32_t> g_trust_polls{4096};

int lamb_params(const dedloc_lamb_cfg *cfg, OptParams &op) {
    if (!cfg) return fail(DEDLOC_ERR_INVALID_ARG, "cfg must not be NULL");
    if (cfg->step == 0) return fail(DEDLOC_ERR_INVALID_ARG, "step must be >= 1");
    memset(&op, 0, sizeof op);
    op.lr = cfg->lr;
    op.wd = cfg->weight_decay;
    op.beta1 = cfg->beta1;
    op.beta2 = cfg->beta2;
    op.omb1 = 1.0f - cfg->beta1;
    op.omb2 = 1.0f - cfg->beta2;
    op.c1 = 1.0f;
    op.c2 = 1.0f;
    if (cfg->bias_correction) {
        op.c1 = (float)(1.0 - pow((double)cfg->beta1, (double)cfg->step));
        op.c2 = (float)(1.0 - pow((double)cfg->beta2, (double)cfg->step));
    }
    op.eps = cfg->eps;
    op.unit_trust = cfg->force_unit_trust ? 1 : 0;
    op.trust_polls = g_trust_polls.load(std::memory_order_relaxed);
    return DEDLOC_OK;
}

int lars_params(const dedloc_lars_cfg *cfg, OptParams &op) {
    if (!cfg) return fail(DEDLOC_ERR_INVALID_ARG, "cfg must not be NULL");
    memset(&op, 0, sizeof op);
    op.lr = cfg->lr;
    op.wd = cfg->weight_decay;
    op.momentum = cfg->momentum;
    op.trust_coef = cfg->trust_coef;
    op.unit_trust = cfg->force_unit_trust ? 1 : 0;
    op.trust_polls = g_trust_polls.load(std::memory_order_relaxed);
    return DEDLOC_OK;
}

// x and the optimizer state (m and v for LAMB, the momentum v for LARS).
// An empty vector (P == 0) reads and writes no element: its buffers may be
// NULL; only the workspace (the per-tensor ratios) is used.
// ws == kNoWs: the caller brings no workspace (the static array is used;
// its size is checked by the caller of this function).
void *const kNoWs = nullptr;

int check_state(int opt, float *x, float *m, float *v, uint64_t P, void *ws, size_t ws_bytes, const Plan &pl,
                bool check_ws = true) {
    if (P > 0 && (!x || !v || (opt == kOptLamb && !m)))
        return fail(DEDLOC_ERR_INVALID_ARG, "parameter and state buffers must not be NULL");
    if (!aligned(x, 16) || !aligned(v, 16) || (m && !aligned(m, 16)))
        return fail(DEDLOC_ERR_ALIGN, "parameter and state buffers must be 16-byte aligned");
    if (!check_ws) return DEDLOC_OK;
    if (!ws || ws_bytes < pl.ws_total)
        return fail(DEDLOC_ERR_WORKSPACE, "workspace of %zu bytes needed (got %zu)", pl.ws_total,
                    ws ? ws_bytes : (size_t)0);
    if (!aligned(ws, 256)) return fail(DEDLOC_ERR_ALIGN, "workspace must be 256-byte aligned");
    return DEDLOC_OK;
}

int grad_src(int32_t codec) {
    return codec == DEDLOC_CODEC_F32 ? kSrcF32 : codec == DEDLOC_CODEC_FP16 ? kSrcFP16 : kSrcI8;
}

// The host's part of the tag of a call's published trust ratios (pass B
// adds the workspace counter that pass A advances): a process-wide
// sequence with a start drawn from the clock and the process id, so that
// workspace contents left by anything else are unlikely to carry it.
uint32_t next_nonce() {
    static std::atomic<uint32_t> ctr{(uint32_t)std::chrono::steady_clock::now().time_since_epoch().count() * 2654435761u ^
                                     (uint32_t)getpid()};
    return ctr.fetch_add(0x9E3779B9u, std::memory_order_relaxed);
}

// Per chunk of tensors: pass A (gradient from src_a) and pass B (LARS reads
// the gradient again from src_b).
int run_opt(int opt, int src_a, int src_b, const Plan &pl, const PeerTable *peers, const GradArgs &ga_a,
            const GradArgs &ga_b, const OptParams &op_in, float *x, float *m, float *v, void *ws,
            float *trust_out, hipStream_t s) {
    static const PeerTable no_peers = {};
    const PeerTable &pt = peers ? *peers : no_peers;
    const int k_a = (opt == kOptLamb ? K_LAMB_A_F32 : K_LARS_A_F32) + std::min(src_a, (int)kSrcPeersFP16);
    const int k_b = opt == kOptLamb ? K_LAMB_B : K_LARS_B;
    const uint32_t nonce = next_nonce();
    OptParams op = op_in;
    const uint32_t cus = pl.one_pass ? cu_count() : 0, groups = cus * kLineGroups;
    op.hold = held_units(cus);
    for (const Chunk &ch : pl.chunks) {
        hipError_t e;
        if (pl.one_pass) {
            const LineWs w = carve_line(pl, ws);
            const uint32_t units = ch.begin[ch.nt];
            RestTable rt;
            memset(&rt, 0, sizeof rt);
            rt.grid_a = std::min(units, groups);
            e = timed(k_a, s, [&] {
                return launch_lamb_a(src_a, ch, rt.grid_a, pt, ga_a, op, x, m, v, w, nonce, trust_out, s);
            });
            if (e != hipSuccess) return hip_fail(e, "optimizer pass A launch");
            for (uint32_t k = 0; k < ch.nt; k++) {
                const uint32_t n = ch.begin[k + 1] - ch.begin[k];
                rt.begin[k] = rt.n_rest;
                if (n > op.hold) rt.n_rest += 2 * (n - op.hold);
            }
            rt.begin[ch.nt] = rt.n_rest;
            const uint32_t n_check = std::max(1u, std::min(cus, units));
            e = timed(k_b, s, [&] { return launch_lamb_b(ch, rt, n_check, op, x, m, v, w, nonce, trust_out, s); });
        } else {
            const TileWs w = carve_tiles(pl, ws);
            e = timed(k_a, s, [&] { return launch_opt_a(opt, src_a, ch, pt, ga_a, op, x, m, v, w, s); });
            if (e != hipSuccess) return hip_fail(e, "optimizer pass A launch");
            e = timed(k_b, s, [&] {
                return launch_opt_b(opt, src_b, pl.nt, ch, ga_b, op, x, m, v, w, nonce, trust_out, s);
            });
        }
        if (e != hipSuccess) return hip_fail(e, "optimizer pass B launch");
    }
    return DEDLOC_OK;
}

// Validation shared by the LAMB and LARS steps.
int prepare_step(int opt, float *x, float *m, float *v, const void *grad, const float *grad_scales,
                 int32_t grad_codec, uint32_t block, uint64_t P, const uint64_t *offsets,
                 const uint8_t *flags, uint32_t n_tensors, void *ws, size_t ws_bytes, Plan &pl) {
    int rc = check_codec(grad_codec, block, true);
    if (rc) return rc;
    rc = check_tensors(P, offsets, n_tensors);
    if (rc) return rc;
    if (!flags) return fail(DEDLOC_ERR_INVALID_ARG, "flags must not be NULL");
    make_plan(opt, false, P, offsets, flags, n_tensors, pl);
    rc = check_state(opt, x, m, v, P, ws, ws_bytes, pl);
    if (rc) return rc;
    if (P == 0) return DEDLOC_OK;
    if (!grad || !aligned(grad, 16)) return fail(DEDLOC_ERR_ALIGN, "grad must be non-NULL and 16-byte aligned");
    if (grad_codec == DEDLOC_CODEC_I8 && (!grad_scales || !aligned(grad_scales, 4)))
        return fail(DEDLOC_ERR_INVALID_ARG, "int8 gradient needs aligned grad_scales");
    return DEDLOC_OK;
}

// Validation shared by the LAMB and LARS rounds.
int prepare_round(int opt, const void *const *peer_codes, const float *const *peer_scales,
                  const uint32_t *counts, uint32_t n_peers, const uint64_t *bounds, uint32_t n_shards,
                  int32_t codec, uint32_t block, void *out_codes, float *out_scales, float *x, float *m,
                  float *v, uint64_t P, const uint64_t *offsets, const uint8_t *flags, uint32_t n_tensors,
                  float *out_mean, const dedloc_local_peer *local, void *ws, size_t ws_bytes,
                  PeerList &peers, Plan &pl, LocalArgs &la, bool check_ws = true) {
    int rc = check_codec(codec, block, false);
    if (rc) return rc;
    rc = build_peers(peer_codes, peer_scales, counts, n_peers, codec, peers, P > 0);
    if (rc) return rc;
    la = LocalArgs{-1, nullptr, nullptr, nullptr};
    if (local) {
        if (local->index >= n_peers || counts[local->index] == 0)
            return fail(DEDLOC_ERR_INVALID_ARG, "the local peer must be one of the peers and hold samples");
        if (P > 0 && (!local->grad || !aligned(local->grad, 16)))
            return fail(DEDLOC_ERR_ALIGN, "the local gradient must be non-NULL and 16-byte aligned");
        for (uint32_t k = 0; k < peers.n(); k++)
            if (peers.index[k] == local->index) la.pos = (int32_t)k;
        la.grad = local->grad;
        la.codes = const_cast<void *>(peer_codes[local->index]);
        la.scales = codec == DEDLOC_CODEC_I8 ? const_cast<float *>(peer_scales[local->index]) : nullptr;
    }
    if (!bounds || n_shards == 0) return fail(DEDLOC_ERR_INVALID_ARG, "bounds must list n_shards >= 1 shards");
    if (bounds[0] != 0 || bounds[n_shards] != P) return fail(DEDLOC_ERR_INVALID_ARG, "shard bounds must tile [0, P)");
    for (uint32_t k = 0; k < n_shards; k++) {
        if (bounds[k + 1] < bounds[k]) return fail(DEDLOC_ERR_INVALID_ARG, "shard bounds decrease at %u", k);
        if (codec == DEDLOC_CODEC_I8 && k > 0 && bounds[k] % block)
            return fail(DEDLOC_ERR_INVALID_ARG, "int8 shard bound %u is not a multiple of the block", k);
    }
    rc = check_tensors(P, offsets, n_tensors);
    if (rc) return rc;
    if (!flags) return fail(DEDLOC_ERR_INVALID_ARG, "flags must not be NULL");
    make_plan(opt, codec == DEDLOC_CODEC_FP16, P, offsets, flags, n_tensors, pl);
    rc = check_state(opt, x, m, v, P, ws, ws_bytes, pl, check_ws);
    if (rc) return rc;
    if (P == 0) return DEDLOC_OK;
    if (!out_codes || !aligned(out_codes, 16)) return fail(DEDLOC_ERR_ALIGN, "out_codes must be non-NULL and 16-byte aligned");
    if (out_mean && !aligned(out_mean, 16)) return fail(DEDLOC_ERR_ALIGN, "out_mean must be 16-byte aligned");
    if (codec == DEDLOC_CODEC_I8 && (!out_scales || !aligned(out_scales, 4)))
        return fail(DEDLOC_ERR_INVALID_ARG, "int8 round needs aligned out_scales");
    return check_chain(peers, out_mean);
}

// The round after validation: the reduce-scatter and gather, then the
// optimizer.  fp16: the codec is elementwise, so every shard's average is the
// same function of the element index and pass A fuses the average of all
// shards (of the last launch's peers, after the earlier ones are summed into
// out_mean).  int8: interior shard bounds sit on block boundaries, so every
// shard's blocks are the vector's blocks and one reduce covers all shards
// before the optimizer reads the gathered message.
int run_round(int opt, const PeerList &peers, int32_t codec, void *out_codes, float *out_scales, float *x,
              float *m, float *v, uint64_t P, const Plan &pl, const OptParams &op, float *trust_out,
              float *out_mean, const LocalArgs &la, void *ws, hipStream_t s) {
    const LocalArgs none = {-1, nullptr, nullptr, nullptr};
    const GradArgs gathered = {out_codes, out_scales, nullptr, nullptr, nullptr, none};
    if (codec == DEDLOC_CODEC_FP16) {
        const uint32_t n = peers.n(), f = last_batch(n);
        int rc = run_reduce(codec, peers, 0, f, false, P, out_codes, nullptr, out_mean, la, s);
        if (rc) return rc;
        const PeerTable pt = table_of(peers, f, n);
        const GradArgs fused = {nullptr, nullptr, (uint16_t *)out_codes, out_mean, out_mean, local_in(la, f, n)};
        const int src = f > 0 ? kSrcPeersFP16Chain : fused.local.pos >= 0 ? kSrcPeersFP16Local : kSrcPeersFP16;
        return run_opt(opt, src, kSrcFP16, pl, &pt, fused, gathered, op, x, m, v, ws, trust_out, s);
    }
    // int8: the local peer's encode stays a launch of its own (folded into
    // the reduce it costs more than it saves: the block encode's wave-wide
    // maximum and divisions lengthen every wave of the reduce)
    if (la.pos >= 0) {
        const hipError_t e = timed(K_ENCODE_I8, s, [&] {
            return launch_encode_i8(la.grad, P, (int8_t *)la.codes, la.scales, s);
        });
        if (e != hipSuccess) return hip_fail(e, "encode launch");
    }
    int rc = run_reduce(codec, peers, 0, peers.n(), true, P, out_codes, out_scales, out_mean, none, s);
    if (rc) return rc;
    return run_opt(opt, kSrcI8, kSrcI8, pl, nullptr, gathered, gathered, op, x, m, v, ws, trust_out, s);
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];  // device address of `scratch` per device (null: not looked up yet)

// The address of this GPU's static scratch array: the current device, which
// `stream` must belong to.  Looked up once per device.
int noalloc_scratch(hipStream_t stream, void **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(DEDLOC_ERR_INVALID_ARG, "device %d is beyond %d", dev, kMaxDevices);
    hipDevice_t sdev = -1;
    e = hipStreamGetDevice(stream, &sdev);
    if (e != hipSuccess) return hip_fail(e, "hipStreamGetDevice");
    if (sdev != dev)
        return fail(DEDLOC_ERR_INVALID_ARG, "the stream belongs to device %d, the current device is %d", (int)sdev, dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!p || !aligned(p, 256)) return fail(DEDLOC_ERR_HIP, "the static scratch array has no usable address");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return DEDLOC_OK;
}

// Group all-reduce layout: m^d slots, m^(d-1) groups per iteration, every
// group message at a 256-byte stride.
struct GroupPlan {
    uint32_t d = 0, slots = 0, groups = 0;
    size_t code_stride = 0, scale_stride = 0;   // bytes, floats
    size_t ws_codes = 0, ws_total = 0;          // two ping-pong sets of group messages
};

int group_plan(uint32_t n, uint32_t m, uint64_t len, int32_t codec, GroupPlan &gp) {
    if (n == 0 || n > DEDLOC_MAX_GROUP_PEERS)
        return fail(DEDLOC_ERR_INVALID_ARG, "n_peers must be in [1, %d]", DEDLOC_MAX_GROUP_PEERS);
    if (m < 2 || m > DEDLOC_MAX_GROUP_SIZE) return fail(DEDLOC_ERR_INVALID_ARG, "group_size must be in [2, %d]", DEDLOC_MAX_GROUP_SIZE);
    uint32_t d = 1;
    uint64_t slots = m;
    while (slots < n) {
        slots *= m;
        d++;
    }
    gp.d = d;
    gp.slots = (uint32_t)slots;
    gp.groups = (uint32_t)(slots / m);
    const size_t cb = codec == DEDLOC_CODEC_FP16 ? 2 : 1;
    gp.code_stride = round_up((size_t)len * cb, 256);
    gp.scale_stride = codec == DEDLOC_CODEC_I8 ? (size_t)((len + DEDLOC_I8_BLOCK - 1) / DEDLOC_I8_BLOCK) : 0;
    const size_t d_prev = d > 1 ? 2 : 0;  // iterations before the last ping-pong between two sets
    gp.ws_codes = d_prev * gp.groups * gp.code_stride;
    gp.ws_total = gp.ws_codes + round_up(d_prev * gp.groups * gp.scale_stride * sizeof(float), 256);
    return DEDLOC_OK;
}

}  // namespace

extern "C" {

int dedloc_version(void) { return 100; }

const char *dedloc_last_error(void) { return g_err.c_str(); }

size_t dedloc_encoded_bytes(int32_t codec, uint32_t block, uint64_t n, uint64_t *n_scales) {
    if (n_scales) *n_scales = 0;
    if (codec == DEDLOC_CODEC_FP16) return (size_t)n * 2;
    if (codec == DEDLOC_CODEC_I8 && block > 0) {
        if (n_scales) *n_scales = (n + block - 1) / block;
        return (size_t)n;
    }
    if (codec == DEDLOC_CODEC_F32) return (size_t)n * 4;
    return 0;
}

int dedloc_partition(uint64_t P, uint32_t n_shards, const uint64_t *weights, uint32_t align,
                     uint64_t *bounds) {
    if (!bounds) return fail(DEDLOC_ERR_INVALID_ARG, "bounds must not be NULL");
    if (n_shards == 0 || align == 0) return fail(DEDLOC_ERR_INVALID_ARG, "n_shards and align must be > 0");
    unsigned __int128 total = 0;
    for (uint32_t k = 0; k < n_shards; k++) total += weights ? weights[k] : 1;
    if (total == 0) return fail(DEDLOC_ERR_INVALID_ARG, "all shard weights are zero");
    const unsigned __int128 denom = total * align;
    unsigned __int128 c = 0;
    bounds[0] = 0;
    for (uint32_t k = 1; k < n_shards; k++) {
        c += weights ? weights[k - 1] : 1;
        bounds[k] = (uint64_t)(((unsigned __int128)P * c / denom) * align);
    }
    bounds[n_shards] = P;
    return DEDLOC_OK;
}

int dedloc_weights(const uint32_t *counts, uint32_t n, float *w) {
    if (!counts || !w || n == 0) return fail(DEDLOC_ERR_INVALID_ARG, "counts/w must be non-NULL, n > 0");
    return compute_weights(counts, n, w);
}

int dedloc_encode(const float *x, uint64_t n, int32_t codec, uint32_t block, void *codes,
                  float *scales, void *stream) {
    int rc = check_codec(codec, block, false);
    if (rc) return rc;
    if (n == 0) return DEDLOC_OK;
    if (!x || !codes) return fail(DEDLOC_ERR_INVALID_ARG, "x and codes must not be NULL");
    if (!aligned(x, 16) || !aligned(codes, 16)) return fail(DEDLOC_ERR_ALIGN, "x and codes must be 16-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e;
    if (codec == DEDLOC_CODEC_FP16) {
        e = timed(K_ENCODE_FP16, s, [&] { return launch_encode_fp16(x, n, (uint16_t *)codes, s); });
    } else {
        if (!scales) return fail(DEDLOC_ERR_INVALID_ARG, "int8 encode needs scales");
        if (!aligned(scales, 4)) return fail(DEDLOC_ERR_ALIGN, "scales must be 4-byte aligned");
        e = timed(K_ENCODE_I8, s, [&] { return launch_encode_i8(x, n, (int8_t *)codes, scales, s); });
    }
    return e == hipSuccess ? DEDLOC_OK : hip_fail(e, "encode launch");
}

int dedloc_decode(const void *codes, const float *scales, uint64_t n, int32_t codec, uint32_t block,
                  float *out, void *stream) {
    int rc = check_codec(codec, block, false);
    if (rc) return rc;
    if (n == 0) return DEDLOC_OK;
    if (!codes || !out) return fail(DEDLOC_ERR_INVALID_ARG, "codes and out must not be NULL");
    if (!aligned(out, 16) || !aligned(codes, 16)) return fail(DEDLOC_ERR_ALIGN, "codes and out must be 16-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e;
    if (codec == DEDLOC_CODEC_FP16) {
        e = timed(K_DECODE_FP16, s, [&] { return launch_decode_fp16((const uint16_t *)codes, n, out, s); });
    } else {
        if (!scales) return fail(DEDLOC_ERR_INVALID_ARG, "int8 decode needs scales");
        if (!aligned(scales, 4)) return fail(DEDLOC_ERR_ALIGN, "scales must be 4-byte aligned");
        e = timed(K_DECODE_I8, s, [&] { return launch_decode_i8((const int8_t *)codes, scales, n, out, s); });
    }
    return e == hipSuccess ? DEDLOC_OK : hip_fail(e, "decode launch");
}

int dedloc_reduce_shard(const void *const *peer_codes, const float *const *peer_scales,
                        const uint32_t *counts, uint32_t n_peers, uint64_t shard_len, int32_t codec,
                        uint32_t block, void *out_codes, float *out_scales, float *out_mean,
                        void *stream) {
    int rc = check_codec(codec, block, false);
    if (rc) return rc;
    PeerList peers;
    rc = build_peers(peer_codes, peer_scales, counts, n_peers, codec, peers, shard_len > 0);
    if (rc) return rc;
    if (shard_len == 0) return DEDLOC_OK;
    if (!out_codes || !aligned(out_codes, 16)) return fail(DEDLOC_ERR_ALIGN, "out_codes must be non-NULL and 16-byte aligned");
    if (out_mean && !aligned(out_mean, 16)) return fail(DEDLOC_ERR_ALIGN, "out_mean must be 16-byte aligned");
    if (codec == DEDLOC_CODEC_I8 && (!out_scales || !aligned(out_scales, 4)))
        return fail(DEDLOC_ERR_INVALID_ARG, "int8 reduce needs aligned out_scales");
    rc = check_chain(peers, out_mean);
    if (rc) return rc;
    const LocalArgs none = {-1, nullptr, nullptr, nullptr};
    return run_reduce(codec, peers, 0, peers.n(), true, shard_len, out_codes, out_scales, out_mean, none,
                      (hipStream_t)stream);
}

size_t dedloc_lamb_workspace_bytes(uint64_t P, const uint64_t *offsets, uint32_t n_tensors) {
    if (check_tensors(P, offsets, n_tensors)) return 0;
    Plan pl;
    make_plan(kOptLamb, false, P, offsets, nullptr, n_tensors, pl);
    return pl.ws_total;
}

int dedloc_workspace_clear(void *ws, size_t ws_bytes, void *stream) {
    if (!ws || !aligned(ws, 4)) return fail(DEDLOC_ERR_INVALID_ARG, "workspace must be non-NULL and 4-byte aligned");
    if (ws_bytes % 4) return fail(DEDLOC_ERR_INVALID_ARG, "ws_bytes must be a multiple of 4 (got %zu)", ws_bytes);
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = timed(K_FILL, s, [&] { return launch_fill_zero(ws, ws_bytes, s); });
    return e == hipSuccess ? DEDLOC_OK : hip_fail(e, "workspace clear launch");
}

int dedloc_lamb_step(float *x, float *m, float *v, const void *grad, const float *grad_scales,
                     int32_t grad_codec, uint32_t block, uint64_t P, const uint64_t *offsets,
                     const uint8_t *flags, uint32_t n_tensors, const dedloc_lamb_cfg *cfg,
                     float *trust_out, void *ws, size_t ws_bytes, void *stream) {
    OptParams op;
    int rc = lamb_params(cfg, op);
    if (rc) return rc;
    Plan pl;
    rc = prepare_step(kOptLamb, x, m, v, grad, grad_scales, grad_codec, block, P, offsets, flags, n_tensors,
                      ws, ws_bytes, pl);
    if (rc) return rc;
    const GradArgs ga = {grad, grad_scales, nullptr, nullptr, nullptr, {-1, nullptr, nullptr, nullptr}};
    const int src = grad_src(grad_codec);
    return run_opt(kOptLamb, src, src, pl, nullptr, ga, ga, op, x, m, v, ws, trust_out, (hipStream_t)stream);
}

int dedloc_lars_step(float *x, float *v, const void *grad, const float *grad_scales, int32_t grad_codec,
                     uint32_t block, uint64_t P, const uint64_t *offsets, const uint8_t *flags,
                     uint32_t n_tensors, const dedloc_lars_cfg *cfg, float *trust_out, void *ws,
                     size_t ws_bytes, void *stream) {
    OptParams op;
    int rc = lars_params(cfg, op);
    if (rc) return rc;
    Plan pl;
    rc = prepare_step(kOptLars, x, nullptr, v, grad, grad_scales, grad_codec, block, P, offsets, flags,
                      n_tensors, ws, ws_bytes, pl);
    if (rc) return rc;
    const GradArgs ga = {grad, grad_scales, nullptr, nullptr, nullptr, {-1, nullptr, nullptr, nullptr}};
    const int src = grad_src(grad_codec);
    return run_opt(kOptLars, src, src, pl, nullptr, ga, ga, op, x, nullptr, v, ws, trust_out, (hipStream_t)stream);
}

int dedloc_round(const void *const *peer_codes, const float *const *peer_scales, const uint32_t *counts,
                 uint32_t n_peers, const uint64_t *bounds, uint32_t n_shards, int32_t codec, uint32_t block,
                 void *out_codes, float *out_scales, float *x, float *m, float *v, uint64_t P,
                 const uint64_t *offsets, const uint8_t *flags, uint32_t n_tensors,
                 const dedloc_lamb_cfg *cfg, float *trust_out, float *out_mean, const dedloc_local_peer *local,
                 void *ws, size_t ws_bytes, void *stream) {
    OptParams op;
    int rc = lamb_params(cfg, op);
    if (rc) return rc;
    PeerList peers;
    Plan pl;
    LocalArgs la;
    rc = prepare_round(kOptLamb, peer_codes, peer_scales, counts, n_peers, bounds, n_shards, codec, block,
                       out_codes, out_scales, x, m, v, P, offsets, flags, n_tensors, out_mean, local, ws, ws_bytes,
                       peers, pl, la);
    if (rc) return rc;
    return run_round(kOptLamb, peers, codec, out_codes, out_scales, x, m, v, P, pl, op, trust_out, out_mean, la,
                     ws, (hipStream_t)stream);
}

int dedloc_round_noalloc(const void *const *peer_codes, const float *const *peer_scales, const uint32_t *counts,
                         uint32_t n_peers, const uint64_t *bounds, uint32_t n_shards, int32_t codec, uint32_t block,
                         void *out_codes, float *out_scales, float *x, float *m, float *v, uint64_t P,
                         const uint64_t *offsets, const uint8_t *flags, uint32_t n_tensors,
                         const dedloc_lamb_cfg *cfg, float *trust_out, float *out_mean,
                         const dedloc_local_peer *local, void *stream) {
    OptParams op;
    int rc = lamb_params(cfg, op);
    if (rc) return rc;
    PeerList peers;
    Plan pl;
    LocalArgs la;
    rc = prepare_round(kOptLamb, peer_codes, peer_scales, counts, n_peers, bounds, n_shards, codec, block,
                       out_codes, out_scales, x, m, v, P, offsets, flags, n_tensors, out_mean, local, kNoWs, 0,
                       peers, pl, la, /*check_ws=*/false);
    if (rc) return rc;
    if (pl.ws_total > DEDLOC_NOALLOC_SCRATCH_BYTES)
        return fail(DEDLOC_ERR_WORKSPACE,
                    "this tensor table needs %zu bytes of workspace, more than the %u of the static scratch array "
                    "(call dedloc_round with a workspace)", pl.ws_total, (unsigned)DEDLOC_NOALLOC_SCRATCH_BYTES);
    void *ws = nullptr;
    rc = noalloc_scratch((hipStream_t)stream, &ws);
    if (rc) return rc;
    return run_round(kOptLamb, peers, codec, out_codes, out_scales, x, m, v, P, pl, op, trust_out, out_mean, la,
                     ws, (hipStream_t)stream);
}

int dedloc_round_lars(const void *const *peer_codes, const float *const *peer_scales, const uint32_t *counts,
                      uint32_t n_peers, const uint64_t *bounds, uint32_t n_shards, int32_t codec,
                      uint32_t block, void *out_codes, float *out_scales, float *x, float *v, uint64_t P,
                      const uint64_t *offsets, const uint8_t *flags, uint32_t n_tensors,
                      const dedloc_lars_cfg *cfg, float *trust_out, float *out_mean,
                      const dedloc_local_peer *local, void *ws, size_t ws_bytes, void *stream) {
    OptParams op;
    int rc = lars_params(cfg, op);
    if (rc) return rc;
    PeerList peers;
    Plan pl;
    LocalArgs la;
    rc = prepare_round(kOptLars, peer_codes, peer_scales, counts, n_peers, bounds, n_shards, codec, block,
                       out_codes, out_scales, x, nullptr, v, P, offsets, flags, n_tensors, out_mean, local, ws,
                       ws_bytes, peers, pl, la);
    if (rc) return rc;
    return run_round(kOptLars, peers, codec, out_codes, out_scales, x, nullptr, v, P, pl, op, trust_out, out_mean,
                     la, ws, (hipStream_t)stream);
}

size_t dedloc_group_allreduce_workspace_bytes(uint32_t n_peers, uint32_t group_size, uint64_t len,
                                              int32_t codec, uint32_t block) {
    if (check_codec(codec, block, false)) return 0;
    GroupPlan gp;
    if (group_plan(n_peers, group_size, len, codec, gp)) return 0;
    return gp.ws_total > 0 ? gp.ws_total : 256;
}

int dedloc_group_allreduce(const void *const *peer_codes, const float *const *peer_scales,
                           const uint32_t *counts, uint32_t n_peers, uint32_t group_size, uint64_t len,
                           int32_t codec, uint32_t block, void *out_codes, float *out_scales,
                           uint32_t *peer_out, uint32_t *n_out, void *ws, size_t ws_bytes, void *stream) {
    int rc = check_codec(codec, block, false);
    if (rc) return rc;
    GroupPlan gp;
    rc = group_plan(n_peers, group_size, len, codec, gp);
    if (rc) return rc;
    if (!peer_codes || !counts) return fail(DEDLOC_ERR_INVALID_ARG, "peer_codes and counts must not be NULL");
    if (codec == DEDLOC_CODEC_I8 && !peer_scales) return fail(DEDLOC_ERR_INVALID_ARG, "int8 messages need peer_scales");
    uint64_t total = 0;
    for (uint32_t i = 0; i < n_peers; i++) total += counts[i];
    if (total == 0) return fail(DEDLOC_ERR_ZERO_WEIGHT, "every peer has zero samples");
    if (total > (1u << 24)) return fail(DEDLOC_ERR_INVALID_ARG, "total sample count exceeds 2^24");
    if (len > 0) {
        for (uint32_t i = 0; i < n_peers; i++) {
            if (counts[i] == 0) continue;  // never read
            if (!peer_codes[i] || !aligned(peer_codes[i], 16))
                return fail(DEDLOC_ERR_ALIGN, "peer %u message must be non-NULL and 16-byte aligned", i);
            if (codec == DEDLOC_CODEC_I8 && (!peer_scales[i] || !aligned(peer_scales[i], 4)))
                return fail(DEDLOC_ERR_ALIGN, "peer %u scales must be non-NULL and 4-byte aligned", i);
        }
    }
    if (!peer_out || !n_out) return fail(DEDLOC_ERR_INVALID_ARG, "peer_out and n_out must not be NULL");
    if (len > 0) {
        if (!out_codes || !aligned(out_codes, 256)) return fail(DEDLOC_ERR_ALIGN, "out_codes must be non-NULL and 256-byte aligned");
        if (codec == DEDLOC_CODEC_I8 && (!out_scales || !aligned(out_scales, 4)))
            return fail(DEDLOC_ERR_INVALID_ARG, "int8 group all-reduce needs aligned out_scales");
        if (gp.ws_total > 0 && (!ws || ws_bytes < gp.ws_total))
            return fail(DEDLOC_ERR_WORKSPACE, "workspace of %zu bytes needed (got %zu)", gp.ws_total, ws ? ws_bytes : (size_t)0);
        if (gp.ws_total > 0 && !aligned(ws, 256)) return fail(DEDLOC_ERR_ALIGN, "workspace must be 256-byte aligned");
    }
    const uint32_t m = group_size;
    std::vector<int64_t> src(gp.slots, -1), nsrc(gp.slots);
    std::vector<uint64_t> cnt(gp.slots, 0), ncnt(gp.slots);
    for (uint32_t i = 0; i < n_peers; i++) cnt[i] = counts[i];
    hipStream_t s = (hipStream_t)stream;
    char *wsc = (char *)ws;
    float *wss = (float *)(wsc + gp.ws_codes);
    GroupTable gt;
    uint32_t copies = 1;
    // launch the groups gathered in gt (one grid row each)
    auto flush = [&]() -> int {
        if (gt.n_groups == 0) return DEDLOC_OK;
        gt.gbegin[gt.n_groups] = gt.pt.n;
        if (len > 0) {
            const ChainArgs ca = {nullptr, nullptr, 1, {-1, nullptr, nullptr, nullptr}, copies, gp.code_stride, gp.scale_stride};
            hipError_t e = codec == DEDLOC_CODEC_FP16
                               ? timed(K_REDUCE_FP16, s, [&] { return launch_reduce_fp16(gt, len, ca, s); })
                               : timed(K_REDUCE_I8, s, [&] { return launch_reduce_i8(gt, len, ca, cu_count(), s); });
            if (e != hipSuccess) return hip_fail(e, "group reduce launch");
        }
        memset(&gt, 0, sizeof gt);
        return DEDLOC_OK;
    };
    // After iteration k the slots that differ only in digits 0..k hold equal
    // messages and counts, so the groups of iteration k that differ only in
    // digits below k (ids equal but for g % lo) average the same messages: the
    // one with g % lo = 0 is computed and stands for all of them.  The last
    // iteration has one such group, written to every output.  64 peers in
    // groups of 4 then move 117 messages instead of 237.
    uint64_t lo = 1;  // m^k, the weight of digit k
    for (uint32_t k = 0; k < gp.d; k++, lo *= m) {
        const bool last = k + 1 == gp.d;
        copies = last ? gp.groups : 1;
        char *dst_c = last ? (char *)out_codes : wsc + (size_t)(k % 2) * gp.groups * gp.code_stride;
        float *dst_s = last ? out_scales : wss + (size_t)(k % 2) * gp.groups * gp.scale_stride;
        const char *prev_c = wsc + (size_t)((k + 1) % 2) * gp.groups * gp.code_stride;
        const float *prev_s = wss + (size_t)((k + 1) % 2) * gp.groups * gp.scale_stride;
        memset(&gt, 0, sizeof gt);
        for (uint32_t g = 0; g < gp.groups; g++) {
            const uint64_t base = (g / lo) * lo * m + (g % lo);
            if (g % lo != 0) {  // the group g - g % lo stands for it
                const uint64_t same = (g / lo) * lo * m;
                for (uint32_t j = 0; j < m; j++) {
                    nsrc[base + j * lo] = nsrc[same] >= 0 ? (int64_t)g : nsrc[same];
                    ncnt[base + j * lo] = ncnt[same];
                }
                continue;
            }
            uint32_t members = 0;
            uint64_t gtotal = 0;
            for (uint32_t j = 0; j < m; j++) {
                gtotal += cnt[base + j * lo];
                members += cnt[base + j * lo] > 0;
            }
            // a launch describes at most kMaxPeers members and kMaxGroups groups
            if (gt.pt.n + members > (uint32_t)kMaxPeers || gt.n_groups == (uint32_t)kMaxGroups) {
                rc = flush();
                if (rc) return rc;
            }
            const uint32_t first = gt.pt.n;
            uint32_t mc[DEDLOC_MAX_GROUP_SIZE];
            uint32_t nm = 0;
            for (uint32_t j = 0; j < m; j++) {
                const uint64_t sl = base + j * lo;
                if (cnt[sl] == 0) continue;
                if (src[sl] < 0) {
                    gt.pt.codes[gt.pt.n] = peer_codes[sl];
                    gt.pt.scales[gt.pt.n] = codec == DEDLOC_CODEC_I8 ? peer_scales[sl] : nullptr;
                } else {
                    gt.pt.codes[gt.pt.n] = prev_c + (size_t)src[sl] * gp.code_stride;
                    gt.pt.scales[gt.pt.n] = codec == DEDLOC_CODEC_I8 ? prev_s + (size_t)src[sl] * gp.scale_stride : nullptr;
                }
                mc[nm++] = (uint32_t)cnt[sl];
                gt.pt.n++;
            }
            if (nm > 0) {
                float w[DEDLOC_MAX_GROUP_SIZE];
                rc = compute_weights(mc, nm, w);
                if (rc) return rc;
                for (uint32_t j = 0; j < nm; j++) gt.pt.w[first + j] = w[j];
            }
            const uint32_t lg = gt.n_groups++;
            gt.gbegin[lg] = first;
            gt.out[lg] = dst_c + (size_t)g * gp.code_stride;
            gt.out_scales[lg] = codec == DEDLOC_CODEC_I8 ? dst_s + (size_t)g * gp.scale_stride : nullptr;
            for (uint32_t j = 0; j < m; j++) {
                const uint64_t sl = base + j * lo;
                nsrc[sl] = gtotal > 0 ? (int64_t)g : -2;
                ncnt[sl] = gtotal;
            }
        }
        rc = flush();
        if (rc) return rc;
        src.swap(nsrc);
        cnt.swap(ncnt);
    }
    for (uint32_t i = 0; i < n_peers; i++) peer_out[i] = src[i] >= 0 ? (uint32_t)src[i] : 0xffffffffu;
    *n_out = gp.groups;
    return DEDLOC_OK;
}

int dedloc_accumulate(float *acc, const void *grad, int32_t grad_codec, uint64_t n, float batch_samples,
                      void *stream) {
    if (grad_codec != DEDLOC_CODEC_F32 && grad_codec != DEDLOC_CODEC_FP16)
        return fail(DEDLOC_ERR_INVALID_ARG, "accumulate takes fp32 or fp16 gradients");
    if (n == 0) return DEDLOC_OK;
    if (!acc || !grad) return fail(DEDLOC_ERR_INVALID_ARG, "acc and grad must not be NULL");
    if (!aligned(acc, 16) || !aligned(grad, 16)) return fail(DEDLOC_ERR_ALIGN, "acc and grad must be 16-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = timed(K_ACCUMULATE, s, [&] {
        return launch_accumulate(acc, grad, grad_codec == DEDLOC_CODEC_FP16, n, batch_samples, s);
    });
    return e == hipSuccess ? DEDLOC_OK : hip_fail(e, "accumulate launch");
}

int dedloc_finalize(float *acc, uint64_t n, uint32_t count, int32_t codec, uint32_t block, void *codes,
                    float *scales, int32_t reset, void *stream) {
    int rc = check_codec(codec, block, false);
    if (rc) return rc;
    if (count == 0) return fail(DEDLOC_ERR_ZERO_WEIGHT, "no samples were accumulated");
    if (count > (1u << 24)) return fail(DEDLOC_ERR_INVALID_ARG, "count %u exceeds 2^24", count);
    if (n == 0) return DEDLOC_OK;
    if (!acc || !codes) return fail(DEDLOC_ERR_INVALID_ARG, "acc and codes must not be NULL");
    if (!aligned(acc, 16) || !aligned(codes, 16)) return fail(DEDLOC_ERR_ALIGN, "acc and codes must be 16-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e;
    if (codec == DEDLOC_CODEC_FP16) {
        e = timed(K_FINALIZE_FP16, s, [&] { return launch_finalize_fp16(acc, n, (float)count, (uint16_t *)codes, reset, s); });
    } else {
        if (!scales || !aligned(scales, 4)) return fail(DEDLOC_ERR_INVALID_ARG, "int8 finalize needs aligned scales");
        e = timed(K_FINALIZE_I8, s, [&] {
            return launch_finalize_i8(acc, n, (float)count, (int8_t *)codes, scales, reset, s);
        });
    }
    return e == hipSuccess ? DEDLOC_OK : hip_fail(e, "finalize launch");
}

int dedloc_profile_begin(uint32_t max_launches) {
    std::lock_guard<std::mutex> lk(g_prof.mu);
    g_prof.on = true;
    g_prof.cap = max_launches;
    g_prof.used = 0;
    g_prof.kind.clear();
    return DEDLOC_OK;
}

int dedloc_profile_end(uint32_t n_kinds, double *total_ms, uint64_t *launches) {
    std::lock_guard<std::mutex> lk(g_prof.mu);
    if (!g_prof.on) return fail(DEDLOC_ERR_INVALID_ARG, "profiling was not started");
    g_prof.on = false;
    for (uint32_t k = 0; k < n_kinds; k++) {
        if (total_ms) total_ms[k] = 0.0;
        if (launches) launches[k] = 0;
    }
    for (size_t i = 0; i < g_prof.used; i++) {
        hipError_t r = hipEventSynchronize(g_prof.ev[2 * i + 1]);
        if (r != hipSuccess) return hip_fail(r, "profile event wait");
        float ms = 0.0f;
        r = hipEventElapsedTime(&ms, g_prof.ev[2 * i], g_prof.ev[2 * i + 1]);
        if (r != hipSuccess) return hip_fail(r, "profile event time");
        const int k = g_prof.kind[i];
        if ((uint32_t)k < n_kinds) {
            if (total_ms) total_ms[k] += ms;
            if (launches) launches[k] += 1;
        }
    }
    g_prof.used = 0;
    return DEDLOC_OK;
}

uint32_t dedloc_test_trust_polls(uint32_t polls) { return g_trust_polls.exchange(polls); }

int dedloc_kernel_kinds(void) { return K_COUNT; }

const char *dedloc_kernel_name(int kind) {
    return (kind >= 0 && kind < K_COUNT) ? kKindNames[kind] : "";
}

}  // extern "C"

// Internal declarations shared by the kernels and the C-ABI layer of
// libdedloc.  Not part of the public interface (include/dedloc.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dedloc {

// Launch-shape tuning (set from measurements on MI355X).
#ifndef DEDLOC_PEER_BATCH
#define DEDLOC_PEER_BATCH 16  // peer loads issued before the first fma
#endif
#ifndef DEDLOC_NT_PEERS
#define DEDLOC_NT_PEERS 1     // non-temporal hint on loads of data read once
#endif
#ifndef DEDLOC_NT_MSG_STORES
#define DEDLOC_NT_MSG_STORES 1  // non-temporal hint on stores of encoded messages
#endif
#ifndef DEDLOC_TRUST_UNROLL
#define DEDLOC_TRUST_UNROLL 8   // tile partials loaded per lane before summing
#endif
#ifndef DEDLOC_I8_BATCH
#define DEDLOC_I8_BATCH 4     // int8 peer messages loaded per batch in the reduce
#endif

constexpr int kWG = 256;               // threads per workgroup: 4 wave64
constexpr int kVec = 8;                // fp32/fp16 elements per lane (16 B of fp16, 2x16 B of fp32)
constexpr int kPeerBatch = DEDLOC_PEER_BATCH;
constexpr int kRow = kWG * kVec;       // elements a workgroup works on at a time

// LAMB in one pass: a persistent grid of kLineGroups workgroups per CU, each
// holding kLineRegs rows in registers and kLineLds rows in LDS (16 KB a row)
// until their tensor's trust ratio is known: 256 CUs hold 768 * 6 rows, 9.4M
// elements.  More workgroups with shorter lines (4 per CU, 2 + 2 rows) and
// fewer with longer ones (2 per CU, 6 + 4) were slower: ALBERT-xlarge's round
// 978 against 1039 and 1081 us, ALBERT-large's 198 against 201 and 223.
constexpr int kLineGroups = 3;
constexpr int kLineRegs = 3;
constexpr int kLineLds = 3;
constexpr int kLineUnits = (kLineRegs + kLineLds) / 2;  // units (two rows) in a line
// peer loads in flight per lane there (4, 8, 16: ALBERT-large with 16 peers 188, 199, 213 us)
constexpr int kLinePeerBatch = 4;
constexpr uint32_t kLineLast = 8;        // workgroups that say that the whole grid runs
constexpr uint32_t kLineShortWait = 48;  // polls of a wait while it does not
constexpr int kMaxPeers = 64;          // peer table lives in the kernel arguments
constexpr int kI8Block = 1024;         // int8 codec block = one wave64 x 16 codes
constexpr int kI8PerLane = 16;
// 60 peers' 8M elements: 4 83.5 us, 8 99.6, 12 90.1, 16 88.9; 4 also leaves room for 8 waves a SIMD
constexpr int kI8Batch = DEDLOC_I8_BATCH;
constexpr int kI8FewWaves = 16;  // where few waves are in flight
constexpr int kChunkTensors = 192;     // tensors described per LAMB launch

// Active peers (counts > 0) in ascending peer order, with their weights.
struct PeerTable {
    const void *codes[kMaxPeers];
    const float *scales[kMaxPeers];
    float w[kMaxPeers];
    uint32_t n;
};

// Groups of peers reduced by one launch (one group for a plain shard
// reduce; the groups of one iteration of the group all-reduce).  Group g
// averages table entries [gbegin[g], gbegin[g+1]) (its members with samples,
// ascending) into out[g] (and out_scales[g] for int8); an empty range
// produces nothing.
constexpr int kMaxGroups = 64;
struct GroupTable {
    PeerTable pt;
    uint32_t gbegin[kMaxGroups + 1];
    void *out[kMaxGroups];
    float *out_scales[kMaxGroups];
    uint32_t n_groups;
};

// The local peer of a round: its fp32 gradient is encoded by the pass that
// averages it (the codes it would have sent are written on the way), at
// position `pos` of the launch's peer table (-1: no local peer here).
struct LocalArgs {
    int32_t pos;
    const float *grad;  // the full vector, indexed like the messages
    void *codes;        // its message (output)
    float *scales;      // int8: its block scales (output)
};

// A reduce over more peers than one table holds is a chain of launches
// through an fp32 running sum (stored exactly between launches, so the fma
// chain is the same as in one pass).  Only a single-group reduce chains, and
// only a single-group fp16 reduce has a local peer.
struct ChainArgs {
    const float *acc_in;  // running sum of the peers before this launch (nullable: start at +0)
    float *acc_out;       // the sum after this launch (the mean after the last launch; nullable)
    int final_pass;       // encode into the group outputs
    LocalArgs local;
    // the encoded average is written `copies` times, at these strides from the
    // group's output (one group; a plain reduce writes it once)
    uint32_t copies;
    uint64_t code_stride, scale_stride;  // bytes, floats
};

// A run of consecutive tensors handled by one optimizer launch (it spans
// fewer than 2^32 elements).  Work items (tiles of one row; units of two in
// LAMB's one pass) never cross a tensor: tensor k of the chunk covers elements
// base + [start[k], start[k+1]) and owns items [begin[k], begin[k+1]).
struct Chunk {
    uint64_t base;                      // absolute offset of the chunk's first element
    uint32_t nt;                        // tensors in this chunk
    uint32_t t0;                        // index of the chunk's first tensor
    uint32_t row_base;                  // rows of the tensors before the chunk
    uint32_t start[kChunkTensors + 1];  // element offsets relative to base
    uint32_t begin[kChunkTensors + 1];
    uint8_t odd_before[kChunkTensors];  // tensors of the chunk before k with an odd number of rows
    uint8_t flags[kChunkTensors];
};

// The rows of a chunk that LAMB's one pass does not hold on chip: those of
// tensor k are workgroups [begin[k], begin[k+1]) of the pass after it, counted
// from its last.
struct RestTable {
    uint32_t begin[kChunkTensors + 1];
    uint32_t n_rest;  // begin[nt]
    uint32_t grid_a;  // workgroups of the one pass
};

// Optimizer applied after the gather.
enum Opt : int {
    kOptLamb = 0,  // Adam moments + layer-wise trust ratio ||x||/||u||
    kOptLars = 1   // momentum SGD + layer-wise rate eta*||x||/(||g|| + wd*||x||)
};

// Hyper-parameters of either optimizer (host-computed constants included).
struct OptParams {
    float lr, wd;
    float beta1, beta2, omb1, omb2, c1, c2, eps;  // LAMB
    float momentum, trust_coef;                   // LARS
    int32_t unit_trust;
    uint32_t trust_polls;  // polls for a tensor's published ratio before doing without it
    uint32_t hold;         // LAMB's pass A holds the last so many units of every tensor on chip
};

// Where the LAMB step takes its gradient from.
enum GradSrc : int {
    kSrcF32 = 0,      // fp32 gradient
    kSrcFP16 = 1,     // fp16 message
    kSrcI8 = 2,       // int8 message + block scales
    kSrcPeersFP16 = 3,      // fused: average the fp16 peer messages, encode, decode
    kSrcPeersFP16Chain = 4, // the same, continuing a running sum of earlier peers (and
                            // with the local peer if the launch holds it)
    kSrcPeersFP16Local = 5  // kSrcPeersFP16 with the local peer's encode
};

struct GradArgs {
    const void *grad;        // kSrcF32 / kSrcFP16 / kSrcI8
    const float *scales;     // kSrcI8
    uint16_t *out_codes;     // kSrcPeersFP16*: gathered encoded average
    float *out_mean;         // kSrcPeersFP16*: fp32 average (nullable)
    const float *acc_in;     // kSrcPeersFP16Chain: running sum of the earlier peers
    LocalArgs local;         // kSrcPeersFP16Chain / kSrcPeersFP16Local
};

struct TileWs {
    double *partials;            // 2 per tile: sum x^2, sum u^2 (LARS: g^2)
    unsigned long long *trust;   // per tensor: (epoch << 32) | bits of r_t, published inside pass B
    uint32_t *epoch;             // the tag of the current launch: advanced by pass A, read by pass B
};

// Every word that another workgroup waits for carries the tag of the launch
// that wrote it.
struct LineWs {
    uint32_t *epoch;             // [0]: read by pass A, advanced by pass B; [1]: pass A's value for pass B
    unsigned long long *state;   // low half: the tag if any tensor of the launch was given up;
                                 // high half: how many of the grid's last kLineLast workgroups run
                                 // (zeroed by pass B; other contents only shorten a launch's waits)
    unsigned long long *part;    // 16 bytes per row: records of partial sums
    unsigned long long *trust;   // per tensor: (tag << 32) | bits of r_t
};

// Launchers (return hipError_t of the launch).
hipError_t launch_encode_fp16(const float *x, uint64_t n, uint16_t *codes, hipStream_t s);
hipError_t launch_decode_fp16(const uint16_t *codes, uint64_t n, float *out, hipStream_t s);
hipError_t launch_encode_i8(const float *x, uint64_t n, int8_t *codes, float *scales, hipStream_t s);
hipError_t launch_decode_i8(const int8_t *codes, const float *scales, uint64_t n, float *out,
                            hipStream_t s);
hipError_t launch_reduce_fp16(const GroupTable &gt, uint64_t len, const ChainArgs &ca, hipStream_t s);
// cus: compute units of the device
hipError_t launch_reduce_i8(const GroupTable &gt, uint64_t len, const ChainArgs &ca, uint32_t cus, hipStream_t s);
hipError_t launch_lamb_a(int src, const Chunk &ch, uint32_t n_groups, const PeerTable &pt, const GradArgs &ga,
                         const OptParams &op, float *x, float *m, float *v, const LineWs &ws, uint32_t nonce,
                         float *trust_out, hipStream_t s);
hipError_t launch_lamb_b(const Chunk &ch, const RestTable &rt, uint32_t n_check, const OptParams &op, float *x, float *m,
                         float *v, const LineWs &ws, uint32_t nonce, float *trust_out, hipStream_t s);
hipError_t launch_opt_a(int opt, int src, const Chunk &ch, const PeerTable &p, const GradArgs &ga,
                        const OptParams &op, float *x, float *m, float *v, const TileWs &ws, hipStream_t s);
hipError_t launch_opt_b(int opt, int src, bool nt, const Chunk &ch, const GradArgs &ga, const OptParams &op, float *x,
                        float *m, float *v, const TileWs &ws, uint32_t nonce, float *trust_out, hipStream_t s);
hipError_t launch_accumulate(float *acc, const void *grad, bool fp16, uint64_t n, float b, hipStream_t s);
hipError_t launch_finalize_fp16(float *acc, uint64_t n, float count, uint16_t *codes, int reset, hipStream_t s);
hipError_t launch_finalize_i8(float *acc, uint64_t n, float count, int8_t *codes, float *scales, int reset,
                              hipStream_t s);
hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s);

}  // namespace dedloc

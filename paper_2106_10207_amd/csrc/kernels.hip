// gfx950 kernels of libdedloc: wire codecs, the weighted shard average, the
// LAMB and LARS step (LAMB in one pass on large vectors, else two passes) and
// local accumulation.
//
// Every kernel streams HBM in 16-byte vectors per lane; nothing here is a
// dense contraction, so there is no MFMA.  Compiled with -ffp-contract=off:
// every fused multiply-add is an explicit fmaf, every other operation rounds
// once, fp32 division and square root are correctly rounded (the HIP
// defaults), so the results are fixed by the definitions in dedloc.h.
#include <algorithm>
#include <tuple>
#include <utility>

#include "dedloc_internal.h"

namespace dedloc {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- helpers

// Loads of data read once (peer messages).
template <typename T>
__device__ __forceinline__ T ld_stream(const T *p) {
    if (DEDLOC_NT_PEERS) return __builtin_nontemporal_load(p);
    return *p;
}
// Stores of encoded messages (read by other peers, not by this kernel).
template <typename T>
__device__ __forceinline__ void st_msg(T *p, T v) {
    if (DEDLOC_NT_MSG_STORES) __builtin_nontemporal_store(v, p);
    else *p = v;
}

__device__ __forceinline__ float h2f(unsigned bits) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
}
__device__ __forceinline__ unsigned f2h(float f) {
    // IEEE round to nearest even, gradual underflow, overflow to infinity
    return __builtin_bit_cast(uint16_t, (_Float16)f);
}

__device__ __forceinline__ void unpack_fp16x8(u32x4 c, float *o) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
        o[2 * i] = h2f(c[i] & 0xffffu);
        o[2 * i + 1] = h2f(c[i] >> 16);
    }
}
__device__ __forceinline__ u32x4 pack_fp16x8(const float *a) {
    u32x4 c;
#pragma unroll
    for (int i = 0; i < 4; i++) c[i] = f2h(a[2 * i]) | (f2h(a[2 * i + 1]) << 16);
    return c;
}

__device__ __forceinline__ float sbyte(unsigned word, int j) {
    return (float)(int)(int8_t)(word >> (8 * j));
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sum of two doubles over the 256-thread block in a fixed tree; thread 0
// gets the result.
__device__ __forceinline__ void block_sum2(double &a, double &b) {
    __shared__ double red[2][kWG / 64];
    a = wave_sum(a);
    b = wave_sum(b);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
        red[0][wave] = a;
        red[1][wave] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
        b = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    }
    __syncthreads();
}

// Lane layout of rows of 2048 fp32 elements, of which a wave works on 512:
// lane l holds elements 4l..4l+3 and 256+4l..256+4l+3 of its wave's 512, so
// that every 16-byte access of the wave covers 1 KB without gaps.  With eight
// consecutive elements per lane (two accesses at a 32-byte stride) a stream of
// 16 bytes read and 12 written per element ran at 5.2 TB/s, with or without
// non-temporal hints; without gaps and with both hints it runs at 5.7 to 6.0
// TB/s (17.7M and 268M elements).
__device__ __forceinline__ uint32_t row_at(int h) {
    return (threadIdx.x & ~63u) * kVec + 256 * h + 4 * (threadIdx.x & 63);
}

// Encode one int8 block held by a wave: 16 values per lane (lanes or values
// past the end hold zero).  Returns the codes packed in a u32x4 and the
// block scale (same on every lane).
//
// The code is rint of the correctly rounded quotient x / s.  It is taken from
// t = x * rcp(s) instead wherever that provably gives the same integer:
// v_rcp_f32 is within 1 ulp of 1/s, so |t - x/s| < 1.5 * 2^-23 * |x/s| and
// |x/s| <= a / fl(a/127) < 127.00001 bound the error by 2.3e-5, and the
// correctly rounded quotient lies within half an ulp (2^-18 below 128) of
// x/s.  When t is farther than 2^-14 from every half-integer, x/s, its
// rounding and t all lie strictly on the same side of every half-integer,
// so rint(t) is the code.  Lanes holding a value closer to a tie, and blocks
// whose scale is outside [2^-100, 2^100] (where rcp could leave the normal
// range), divide.
__device__ __forceinline__ u32x4 encode_i8_wave(const float *val, float &scale) {
    float a = 0.0f;
#pragma unroll
    for (int j = 0; j < kI8PerLane; j++) a = fmaxf(a, fabsf(val[j]));
    a = wave_max(a);
    const float s = a / 127.0f;
    scale = s;
    u32x4 c = {0u, 0u, 0u, 0u};
    if (s != 0.0f) {  // s == 0: an all-zero block, or a / 127 underflowed; every code is 0
        float q[kI8PerLane];
        bool divide = !(s >= 0x1p-100f && s <= 0x1p100f);  // wave-uniform
        if (!divide) {
            const float y = __builtin_amdgcn_rcpf(s);
#pragma unroll
            for (int j = 0; j < kI8PerLane; j++) {
                const float t = val[j] * y;
                q[j] = rintf(t);
                divide |= fabsf(t - q[j]) > 0.5f - 0x1p-14f;  // t - rint(t) is exact
            }
        }
        if (divide) {
#pragma unroll
            for (int j = 0; j < kI8PerLane; j++) q[j] = rintf(val[j] / s);
        }
#pragma unroll
        for (int j = 0; j < kI8PerLane; j++) {
            const float qc = fminf(fmaxf(q[j], -127.0f), 127.0f);
            c[j >> 2] |= ((unsigned)(int)qc & 0xffu) << (8 * (j & 3));
        }
    }
    return c;
}

// -------------------------------------------------------------- fp16 codec

__global__ __launch_bounds__(kWG) void encode_fp16_kernel(const float *__restrict__ x, uint64_t n,
                                                          uint16_t *__restrict__ codes) {
    const uint64_t row = (uint64_t)blockIdx.x * kRow;
    if (row + kRow <= n) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const f32x4 a = ld_stream((const f32x4 *)(x + row + row_at(h)));
            // plain stores (non-temporal / plain): with the message read next, here
            // decoded, 8M elements 18.7 / 13.2 us, 17.7M 37.1 / 33.8, 60M 116.8 / 106.4;
            // alone 6.9 / 7.4, 15.6 / 17.8, 100M 90.4 / 86.3
            *(u32x2 *)(codes + row + row_at(h)) = u32x2{f2h(a[0]) | (f2h(a[1]) << 16), f2h(a[2]) | (f2h(a[3]) << 16)};
        }
    } else {
        for (uint64_t e = row + threadIdx.x; e < n; e += kWG) codes[e] = (uint16_t)f2h(x[e]);
    }
}

// NT: non-temporal stores of the decoded vector, from these sizes on.  A small
// vector is found in the L2s by whoever reads it next (int8 decode, then accumulate,
// plain / non-temporal: 65k elements 3.96 / 4.06 us, 262k 4.28 / 4.46, 1M 6.42 / 6.66,
// 1.5M 8.00 / 8.18, 2M 9.40 / 9.25; fp16 1M 4.85 / 4.87, 1.5M 5.57 / 5.51, 2M 6.63 /
// 6.31); a large one leaves them room for the message and the reader's other data
// (8M int8: alone 7.70 / 5.94, after the encode 16.5 / 12.9, before an accumulate 22.6 /
// 22.5; 17.7M fp16: 17.1 / 16.7, 37.1 / 33.8, 48.6 / 49.1).  A reader that writes as much
// again into a third buffer loses by it where the Infinity Cache would have held the
// vector (40M fp16: 82.8 / 94.1).
constexpr uint64_t kNtDecodeFp16 = 1ull << 20, kNtDecodeI8 = 1ull << 21;
template <bool NT>
__device__ __forceinline__ void st_decoded(f32x4 *p, f32x4 v) {
    if (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

template <bool NT>
__global__ __launch_bounds__(kWG) void decode_fp16_kernel(const uint16_t *__restrict__ codes, uint64_t n,
                                                          float *__restrict__ out) {
    const uint64_t row = (uint64_t)blockIdx.x * kRow;
    if (row + kRow <= n) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const u32x2 c = *(const u32x2 *)(codes + row + row_at(h));
            st_decoded<NT>((f32x4 *)(out + row + row_at(h)),
                           f32x4{h2f(c[0] & 0xffffu), h2f(c[0] >> 16), h2f(c[1] & 0xffffu), h2f(c[1] >> 16)});
        }
    } else {
        for (uint64_t e = row + threadIdx.x; e < n; e += kWG) out[e] = h2f(codes[e]);
    }
}

// -------------------------------------------------------------- int8 codec
// One wave per 1024-element block, 16 elements per lane.  In the standalone
// codec kernels lane l holds elements 256*q + 4*l + r (q, r in 0..3) of its
// block, so that every 16-byte fp32 access of the wave covers 1 KB without
// gaps (the block maximum and the per-element codes do not depend on which
// lane holds which element).

__device__ __forceinline__ uint64_t i8_lane_base(uint64_t blk) { return blk * kI8Block + 4 * (threadIdx.x & 63); }
#define I8_ELEM(b0, q, r) ((b0) + 256 * (q) + (r))

// The lane's 16 fp32 values of block blk (zero past n).
__device__ __forceinline__ void load_i8_lane(const float *__restrict__ x, uint64_t n, uint64_t blk, float *val) {
    const uint64_t b0 = i8_lane_base(blk);
    if ((blk + 1) * kI8Block <= n) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const f32x4 a = ld_stream((const f32x4 *)(x + I8_ELEM(b0, q, 0)));
            val[4 * q] = a[0]; val[4 * q + 1] = a[1]; val[4 * q + 2] = a[2]; val[4 * q + 3] = a[3];
        }
    } else {
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const uint64_t e = I8_ELEM(b0, q, r);
                val[4 * q + r] = e < n ? x[e] : 0.0f;
            }
    }
}

// Store the lane's 16 codes of block blk (those below n) and the scale.
__device__ __forceinline__ void store_i8_lane(int8_t *__restrict__ codes, float *__restrict__ scales, uint64_t n,
                                              uint64_t blk, u32x4 c, float s) {
    const uint64_t b0 = i8_lane_base(blk);
    if ((blk + 1) * kI8Block <= n) {
#pragma unroll
        // plain stores: with a non-temporal hint the reduce that reads this
        // message next ran 40 us slower on ALBERT-xlarge
        for (int q = 0; q < 4; q++) *(unsigned *)(codes + I8_ELEM(b0, q, 0)) = c[q];
    } else {
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const uint64_t e = I8_ELEM(b0, q, r);
                if (e < n) codes[e] = (int8_t)(c[q] >> (8 * r));
            }
    }
    if ((threadIdx.x & 63) == 0) scales[blk] = s;
}

__global__ __launch_bounds__(kWG) void encode_i8_kernel(const float *__restrict__ x, uint64_t n,
                                                        int8_t *__restrict__ codes,
                                                        float *__restrict__ scales) {
    const uint64_t blk = (uint64_t)blockIdx.x * (kWG / 64) + (threadIdx.x >> 6);
    if (blk * kI8Block >= n) return;  // whole wave past the end
    float val[kI8PerLane];
    load_i8_lane(x, n, blk, val);
    float s;
    const u32x4 c = encode_i8_wave(val, s);
    store_i8_lane(codes, scales, n, blk, c, s);
}

template <bool NT>
__global__ __launch_bounds__(kWG) void decode_i8_kernel(const int8_t *__restrict__ codes,
                                                        const float *__restrict__ scales, uint64_t n,
                                                        float *__restrict__ out) {
    const uint64_t blk = (uint64_t)blockIdx.x * (kWG / 64) + (threadIdx.x >> 6);
    if (blk * kI8Block >= n) return;  // whole wave past the end
    const float s = scales[blk];
    const uint64_t b0 = i8_lane_base(blk);
    if ((blk + 1) * kI8Block <= n) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const unsigned c = *(const unsigned *)(codes + I8_ELEM(b0, q, 0));
            st_decoded<NT>((f32x4 *)(out + I8_ELEM(b0, q, 0)),
                       f32x4{sbyte(c, 0) * s, sbyte(c, 1) * s, sbyte(c, 2) * s, sbyte(c, 3) * s});
        }
    } else {
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const uint64_t e = I8_ELEM(b0, q, r);
                if (e < n) out[e] = (float)codes[e] * s;
            }
    }
}

// ------------------------------------------------------------- the reducer
// mean[e] = sum over the active peers of a group (ascending) of
// w_p * dec_p[e], one fma per peer starting from +0.  A launch reduces every
// group of a GroupTable: grid row blockIdx.y is the group.

// Running sums of eight consecutive elements: from acc_in, or +0.
__device__ __forceinline__ void init8(const float *acc_in, uint64_t e0, float *acc) {
    if (acc_in) {
        const f32x4 a = *(const f32x4 *)(acc_in + e0), b = *(const f32x4 *)(acc_in + e0 + 4);
        acc[0] = a[0]; acc[1] = a[1]; acc[2] = a[2]; acc[3] = a[3];
        acc[4] = b[0]; acc[5] = b[1]; acc[6] = b[2]; acc[7] = b[3];
    } else {
#pragma unroll
        for (int i = 0; i < 8; i++) acc[i] = 0.0f;
    }
}

// Eight consecutive fp16 elements starting at e0 (all in range), peers
// [p_lo, p_hi) of the table, added to the running sums in acc.
template <int B>  // peer loads kept in flight per lane
__device__ __forceinline__ void reduce_fp16x8(const PeerTable &pt, uint32_t p_lo, uint32_t p_hi,
                                              uint64_t e0, float *acc) {
    for (uint32_t p0 = p_lo; p0 < p_hi; p0 += B) {
        u32x4 c[B];
#pragma unroll
        for (int j = 0; j < B; j++)
            if (p0 + j < p_hi) c[j] = ld_stream((const u32x4 *)((const uint16_t *)pt.codes[p0 + j] + e0));
#pragma unroll
        for (int j = 0; j < B; j++) {
            if (p0 + j < p_hi) {
                const float w = pt.w[p0 + j];
                float d[8];
                unpack_fp16x8(c[j], d);
#pragma unroll
                for (int i = 0; i < 8; i++) acc[i] = fmaf(w, d[i], acc[i]);
            }
        }
    }
}

__device__ __forceinline__ float reduce_fp16_one(const PeerTable &pt, uint32_t p_lo, uint32_t p_hi,
                                                 uint64_t e, float acc) {
    for (uint32_t p = p_lo; p < p_hi; p++)
        acc = fmaf(pt.w[p], h2f(((const uint16_t *)pt.codes[p])[e]), acc);
    return acc;
}

// Peers [0, n) of the table added to acc, the peer at lp (< n) being the
// local one: its eight fp32 values are encoded, the codes stored as its
// message and their decoded values averaged like any peer's.  (Issuing the
// next peers' loads before the local peer's values are used measured the
// same, and keeping the local loads inside a peer batch costs registers.)
// NT: the gradient's loads carry the non-temporal hint.  Chosen per kernel that
// calls it, by times per round with the hint / without, three sets of buffers
// in turn and the same set again and again.  LAMB's pass A, ResNet-50: 32 peers
// 500 / 503 and 437 / 462 us, 16 peers 335 / 339 and 285 / 305 (three sets: 6M
// elements in 60 tensors 56.0 / 57.5, 2M in 30 26.0 / 26.1; with few tensors the
// other way round, 2.8M in 2 33.9 / 32.9, 5M in 3 46.5 / 46.1); LARS' pass A,
// 32 peers: 415 / 418 and 413 / 399; reduce_fp16_kernel, ALBERT-large's round of
// 100 peers: 798 / 810 and 783 / 771, ResNet-50's 1220 / 1214 and 1153 / 1177.
// lamb_a_kernel, which has 4 peer loads in flight and not 16: ALBERT-large, the
// same set again, 207 / 198 (the two halves of each 32 bytes are fetched apart).
template <int B, bool NT>
__device__ __forceinline__ void reduce_fp16x8_local(const PeerTable &pt, uint32_t n, uint32_t lp,
                                                    const LocalArgs &la, uint64_t e0, float *acc) {
    reduce_fp16x8<B>(pt, 0, lp, e0, acc);
    const f32x4 *q = (const f32x4 *)(la.grad + e0);
    const f32x4 ga = NT ? ld_stream(q) : q[0], gb = NT ? ld_stream(q + 1) : q[1];
    const float v[8] = {ga[0], ga[1], ga[2], ga[3], gb[0], gb[1], gb[2], gb[3]};
    const u32x4 lc = pack_fp16x8(v);
    st_msg((u32x4 *)((uint16_t *)la.codes + e0), lc);
    float d[8];
    unpack_fp16x8(lc, d);
    const float w = pt.w[lp];
#pragma unroll
    for (int i = 0; i < 8; i++) acc[i] = fmaf(w, d[i], acc[i]);
    reduce_fp16x8<B>(pt, lp + 1, n, e0, acc);
}

__device__ __forceinline__ float reduce_fp16_one_local(const PeerTable &pt, uint32_t n, uint32_t lp,
                                                       const LocalArgs &la, uint64_t e, float acc) {
    acc = reduce_fp16_one(pt, 0, lp, e, acc);
    const unsigned c = f2h(la.grad[e]);
    ((uint16_t *)la.codes)[e] = (uint16_t)c;
    acc = fmaf(pt.w[lp], h2f(c), acc);
    return reduce_fp16_one(pt, lp + 1, n, e, acc);
}

// B: peer loads per batch (small groups take a small batch, which keeps
// registers and so more waves in flight).  Only the full batch handles a
// local peer.
template <int B>
__global__ __launch_bounds__(kWG) void reduce_fp16_kernel(const GroupTable gt, uint64_t len,
                                                          const ChainArgs ca) {
    const uint32_t g = blockIdx.y;
    const uint32_t p_lo = gt.gbegin[g], p_hi = gt.gbegin[g + 1];
    if (p_lo == p_hi) return;  // a group without samples produces nothing
    uint16_t *out = (uint16_t *)gt.out[g];
    float *mean = ca.acc_out;  // may alias ca.acc_in (same element, same lane)
    const uint64_t e0 = ((uint64_t)blockIdx.x * kWG + threadIdx.x) * kVec;
    const bool local = B == kPeerBatch && ca.local.pos >= 0;  // single group: p_lo = 0
    if (e0 + kVec <= len) {
        float acc[8];
        init8(ca.acc_in, e0, acc);
        if (local) reduce_fp16x8_local<B, true>(gt.pt, p_hi, ca.local.pos, ca.local, e0, acc);
        else reduce_fp16x8<B>(gt.pt, p_lo, p_hi, e0, acc);
        if (ca.final_pass) {
            const u32x4 c = pack_fp16x8(acc);
            for (uint32_t k = 0; k < ca.copies; k++) *(u32x4 *)((char *)(out + e0) + k * ca.code_stride) = c;
        }
        if (mean) {
            *(f32x4 *)(mean + e0) = f32x4{acc[0], acc[1], acc[2], acc[3]};
            *(f32x4 *)(mean + e0 + 4) = f32x4{acc[4], acc[5], acc[6], acc[7]};
        }
    } else {
        for (uint64_t e = e0; e < len; e++) {
            const float a0 = ca.acc_in ? ca.acc_in[e] : 0.0f;
            const float a = local ? reduce_fp16_one_local(gt.pt, p_hi, ca.local.pos, ca.local, e, a0)
                                  : reduce_fp16_one(gt.pt, p_lo, p_hi, e, a0);
            if (ca.final_pass)
                for (uint32_t k = 0; k < ca.copies; k++) *(uint16_t *)((char *)(out + e) + k * ca.code_stride) = (uint16_t)f2h(a);
            if (mean) mean[e] = a;
        }
    }
}

// Codes (16 per lane) and block scales of block blk of peers
// [p0, min(p0 + B, p_hi)); `full` if all 16 elements of the lane are in range.
template <int B>
__device__ __forceinline__ void load_i8_batch(const PeerTable &pt, uint32_t p0, uint32_t p_hi, uint64_t blk,
                                              uint64_t e0, uint64_t len, bool full, u32x4 *c, float *s) {
#pragma unroll
    for (int j = 0; j < B; j++) {
        if (p0 + j < p_hi) {
            const int8_t *src = (const int8_t *)pt.codes[p0 + j];
            s[j] = pt.scales[p0 + j][blk];
            if (full) {
                c[j] = ld_stream((const u32x4 *)(src + e0));
            } else {
                c[j] = u32x4{0u, 0u, 0u, 0u};
                for (int k = 0; k < kI8PerLane; k++)
                    if (e0 + k < len) c[j][k >> 2] |= ((unsigned)(uint8_t)src[e0 + k]) << (8 * (k & 3));
            }
        }
    }
}

template <int B>
__device__ __forceinline__ void fma_i8_batch(const PeerTable &pt, uint32_t p0, uint32_t p_hi, const u32x4 *c,
                                             const float *s, float *acc) {
#pragma unroll
    for (int j = 0; j < B; j++) {
        if (p0 + j < p_hi) {
            const float w = pt.w[p0 + j];
#pragma unroll
            for (int k = 0; k < kI8PerLane; k++) {
                const float d = sbyte(c[j][k >> 2], k & 3) * s[j];
                acc[k] = fmaf(w, d, acc[k]);
            }
        }
    }
}

// Peers [p_lo, p_hi) of the table added to the lane's 16 running sums of
// block blk (elements e0..).
template <int B>  // peer loads issued before the batch's fmas
__device__ __forceinline__ void reduce_i8_range(const PeerTable &pt, uint32_t p_lo, uint32_t p_hi, uint64_t blk,
                                                uint64_t e0, uint64_t len, bool full, float *acc) {
    for (uint32_t p0 = p_lo; p0 < p_hi; p0 += B) {
        u32x4 c[B];
        float s[B];
        load_i8_batch<B>(pt, p0, p_hi, blk, e0, len, full, c, s);
        fma_i8_batch<B>(pt, p0, p_hi, c, s, acc);
    }
}

// One wave per 1024-element block; lane holds 16 elements.  B as for
// reduce_fp16_kernel.
template <int B>
__global__ __launch_bounds__(kWG) void reduce_i8_kernel(const GroupTable gt, uint64_t len,
                                                        const ChainArgs ca) {
    const uint32_t g = blockIdx.y;
    const uint32_t p_lo = gt.gbegin[g], p_hi = gt.gbegin[g + 1];
    if (p_lo == p_hi) return;  // a group without samples produces nothing
    int8_t *out = (int8_t *)gt.out[g];
    float *out_scales = gt.out_scales[g];
    const PeerTable &pt = gt.pt;
    const uint64_t blk = (uint64_t)blockIdx.x * (kWG / 64) +
                         (uint64_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blk * kI8Block >= len) return;  // whole wave past the end
    const uint64_t e0 = blk * kI8Block + (threadIdx.x & 63) * kI8PerLane;
    const bool full = e0 + kI8PerLane <= len;
    float *mean = ca.acc_out;  // may alias ca.acc_in (same element, same lane)
    float acc[kI8PerLane];
    if (ca.acc_in && full) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const f32x4 a = *(const f32x4 *)(ca.acc_in + e0 + 4 * q);
            acc[4 * q] = a[0]; acc[4 * q + 1] = a[1]; acc[4 * q + 2] = a[2]; acc[4 * q + 3] = a[3];
        }
    } else {
#pragma unroll
        for (int j = 0; j < kI8PerLane; j++) acc[j] = (ca.acc_in && e0 + j < len) ? ca.acc_in[e0 + j] : 0.0f;
    }
    reduce_i8_range<B>(pt, p_lo, p_hi, blk, e0, len, full, acc);
    if (mean) {
        if (full) {
#pragma unroll
            for (int q = 0; q < 4; q++)
                *(f32x4 *)(mean + e0 + 4 * q) = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        } else {
            for (int k = 0; k < kI8PerLane; k++)
                if (e0 + k < len) mean[e0 + k] = acc[k];
        }
    }
    if (!ca.final_pass) return;  // wave-uniform
    float s;
    const u32x4 c = encode_i8_wave(acc, s);  // out-of-range lanes hold 0
    for (uint32_t n = 0; n < ca.copies; n++, out += ca.code_stride, out_scales += ca.scale_stride) {
        if (full) {
            *(u32x4 *)(out + e0) = c;
        } else {
            for (int k = 0; k < kI8PerLane; k++)
                if (e0 + k < len) out[e0 + k] = (int8_t)(c[k >> 2] >> (8 * (k & 3)));
        }
        if ((threadIdx.x & 63) == 0) out_scales[blk] = s;
    }
}

// ------------------------------------------------------- LAMB and LARS

__device__ __forceinline__ float lamb_dir(float mn, float vn, float x, float lam,
                                          const OptParams &op) {
    const float mh = mn / op.c1;
    const float vh = vn / op.c2;
    return mh / (sqrtf(vh) + op.eps) + lam * x;
}

// Tensor of tile or unit b of a chunk: the largest k with begin[k] <= b (empty
// tensors own none and are skipped).  All values are wave-uniform.
__device__ __forceinline__ uint32_t chunk_tensor(const Chunk &ch, uint32_t b) {
    uint32_t lo = 0, hi = ch.nt;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (ch.begin[mid] <= b) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Gradient of the elements [e0, e0+cnt), cnt <= 8, for source SRC (NT: as
// for reduce_fp16x8_local).
template <int SRC, int B, bool NT>
__device__ __forceinline__ void load_grad(const GradArgs &ga, const PeerTable &pt, uint64_t e0,
                                          int cnt, float *g) {
    if (cnt == kVec) {
        if (SRC == kSrcF32) {
            const f32x4 a = *(const f32x4 *)((const float *)ga.grad + e0);
            const f32x4 b = *(const f32x4 *)((const float *)ga.grad + e0 + 4);
            g[0] = a[0]; g[1] = a[1]; g[2] = a[2]; g[3] = a[3];
            g[4] = b[0]; g[5] = b[1]; g[6] = b[2]; g[7] = b[3];
        } else if (SRC == kSrcFP16) {
            unpack_fp16x8(*(const u32x4 *)((const uint16_t *)ga.grad + e0), g);
        } else if (SRC == kSrcI8) {
            const u32x2 c = *(const u32x2 *)((const int8_t *)ga.grad + e0);
            const float s = ga.scales[e0 / kI8Block];
#pragma unroll
            for (int j = 0; j < 8; j++) g[j] = sbyte(c[j >> 2], j & 3) * s;
        } else {
            float acc[8];
            init8(SRC == kSrcPeersFP16Chain ? ga.acc_in : nullptr, e0, acc);
            if (SRC != kSrcPeersFP16 && ga.local.pos >= 0) reduce_fp16x8_local<B, NT>(pt, pt.n, ga.local.pos, ga.local, e0, acc);
            else reduce_fp16x8<B>(pt, 0, pt.n, e0, acc);
            const u32x4 c = pack_fp16x8(acc);
            st_msg((u32x4 *)(ga.out_codes + e0), c);
            if (ga.out_mean) {
                *(f32x4 *)(ga.out_mean + e0) = f32x4{acc[0], acc[1], acc[2], acc[3]};
                *(f32x4 *)(ga.out_mean + e0 + 4) = f32x4{acc[4], acc[5], acc[6], acc[7]};
            }
            unpack_fp16x8(c, g);
        }
    } else {
        for (int j = 0; j < kVec; j++) {
            if (j >= cnt) {
                g[j] = 0.0f;
                continue;
            }
            const uint64_t e = e0 + j;
            if (SRC == kSrcF32) {
                g[j] = ((const float *)ga.grad)[e];
            } else if (SRC == kSrcFP16) {
                g[j] = h2f(((const uint16_t *)ga.grad)[e]);
            } else if (SRC == kSrcI8) {
                g[j] = (float)((const int8_t *)ga.grad)[e] * ga.scales[e / kI8Block];
            } else {
                const float a0 = SRC == kSrcPeersFP16Chain ? ga.acc_in[e] : 0.0f;
                const float a = SRC != kSrcPeersFP16 && ga.local.pos >= 0
                                    ? reduce_fp16_one_local(pt, pt.n, ga.local.pos, ga.local, e, a0)
                                    : reduce_fp16_one(pt, 0, pt.n, e, a0);
                const unsigned c = f2h(a);
                ga.out_codes[e] = (uint16_t)c;
                if (ga.out_mean) ga.out_mean[e] = a;
                g[j] = h2f(c);
            }
        }
    }
}

// Eight elements per lane, of which cnt exist.  NT: non-temporal, for state
// that is not read again before the caches have turned over.
template <bool NT>
__device__ __forceinline__ void load8(const float *p, uint64_t e0, int cnt, float *o) {
    if (cnt == kVec) {
        const f32x4 *q = (const f32x4 *)(p + e0);
        const f32x4 a = NT ? __builtin_nontemporal_load(q) : q[0], b = NT ? __builtin_nontemporal_load(q + 1) : q[1];
        o[0] = a[0]; o[1] = a[1]; o[2] = a[2]; o[3] = a[3];
        o[4] = b[0]; o[5] = b[1]; o[6] = b[2]; o[7] = b[3];
    } else {
#pragma unroll
        for (int j = 0; j < kVec; j++) o[j] = j < cnt ? p[e0 + j] : 0.0f;
    }
}

template <bool NT>
__device__ __forceinline__ void store8(float *p, uint64_t e0, int cnt, const float *o) {
    if (cnt == kVec) {
        f32x4 *q = (f32x4 *)(p + e0);
        const f32x4 a = {o[0], o[1], o[2], o[3]}, b = {o[4], o[5], o[6], o[7]};
        if (NT) {
            __builtin_nontemporal_store(a, q);
            __builtin_nontemporal_store(b, q + 1);
        } else {
            q[0] = a;
            q[1] = b;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kVec; j++)
            if (j < cnt) p[e0 + j] = o[j];
    }
}

__device__ __forceinline__ int count8(uint64_t e0, uint64_t t_hi) {
    return e0 >= t_hi ? 0 : (int)(t_hi - e0 < (uint64_t)kVec ? t_hi - e0 : (uint64_t)kVec);
}

// The ratio of a tensor from its sums (r = 1 when disabled or a norm is 0).
//   LAMB: r = ||x|| / ||u||;  LARS: r = eta*||x|| / (||g|| + lambda*||x||).
template <int OPT>
__device__ __forceinline__ float trust_ratio(uint8_t flags, const OptParams &op, double a0, double a1) {
    const double X = sqrt(a0), Y = sqrt(a1);
    float r = 1.0f;
    if (!op.unit_trust && (flags & 2u) && X > 0.0 && Y > 0.0) {
        if (OPT == kOptLamb) {
            r = (float)(X / Y);
        } else {
            const double lam = (flags & 1u) ? (double)op.wd : 0.0;
            r = (float)((double)op.trust_coef * X / (Y + lam * X));
        }
    }
    return r;
}

// --------------------------------------------- the optimizer in two passes
// Pass A: gradient (optionally the fused average), for LAMB the new moments,
// and the per-tile sums of x^2 and u^2 (LARS: g^2), in fp64 with a fixed tree
// inside the tile; pass B: the ratios and the update, from memory again.
// NT (LARS's pass B): non-temporal accesses for state that the 256 MB Infinity
// Cache does not keep from one call to the next (ResNet-50, 32 peers: 419 ->
// 412 us, 40M elements 232 -> 222; on 6M, which it keeps, 31.2 -> 33.6: the
// caller chooses by size).  LAMB's passes were slower with them (60M elements
// in 400 tensors 606 -> 631 us: pass B finds part of x, m', v' in the cache).
template <int SRC, int OPT>
__global__ __launch_bounds__(kWG) void opt_a_kernel(const Chunk ch, const PeerTable pt, const GradArgs ga,
                                                    const OptParams op, const float *__restrict__ x,
                                                    float *__restrict__ m, float *__restrict__ v, TileWs ws) {
    const uint32_t b = blockIdx.x;
    const uint32_t k = chunk_tensor(ch, b);
    const uint64_t t_lo = ch.base + ch.start[k], t_hi = ch.base + ch.start[k + 1];
    const uint32_t tile = b - ch.begin[k];
    const float lam = (ch.flags[k] & 1u) ? op.wd : 0.0f;
    double s0 = 0.0, s1 = 0.0;
    const uint64_t e0 = t_lo + (uint64_t)tile * kRow + threadIdx.x * kVec;
    const int cnt = count8(e0, t_hi);
    if (cnt > 0) {
        float g[8], xv[8];
        load8<false>(x, e0, cnt, xv);
        if (OPT == kOptLamb) {
            float mv[8], vv[8];
            load8<false>(m, e0, cnt, mv);
            load8<false>(v, e0, cnt, vv);
            load_grad<SRC, kPeerBatch, OPT == kOptLamb>(ga, pt, e0, cnt, g);
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const float mn = fmaf(op.beta1, mv[j], op.omb1 * g[j]);
                const float vn = fmaf(op.beta2, vv[j], op.omb2 * (g[j] * g[j]));
                const float u = lamb_dir(mn, vn, xv[j], lam, op);
                mv[j] = mn;
                vv[j] = vn;
                if (j < cnt) {
                    s0 += (double)xv[j] * (double)xv[j];
                    s1 += (double)u * (double)u;
                }
            }
            store8<false>(m, e0, cnt, mv);
            store8<false>(v, e0, cnt, vv);
        } else {
            load_grad<SRC, kPeerBatch, OPT == kOptLamb>(ga, pt, e0, cnt, g);
#pragma unroll
            for (int j = 0; j < 8; j++) {
                if (j < cnt) {
                    s0 += (double)xv[j] * (double)xv[j];
                    s1 += (double)g[j] * (double)g[j];
                }
            }
        }
    }
    block_sum2(s0, s1);
    if (threadIdx.x == 0) {
        ws.partials[2 * (uint64_t)(ch.row_base + b)] = s0;
        ws.partials[2 * (uint64_t)(ch.row_base + b) + 1] = s1;
        // a fresh tag for the ratios pass B publishes (the only access to
        // this word during the launch; pass B reads it after the launch)
        if (b == 0) ws.epoch[0] = ws.epoch[0] + 1u;
    }
}

// Sums over tensor k of the chunk of its tile partials (x^2, and u^2 or
// g^2), in a fixed order: lane-strided, then a fixed tree.  Every thread of
// the workgroup calls it; thread 0 gets the sums.
__device__ __forceinline__ void tensor_sums(const Chunk &ch, const TileWs &ws, uint32_t k, double &a0, double &a1) {
    const uint32_t first = ch.row_base + ch.begin[k];
    const uint32_t ntiles = ch.begin[k + 1] - ch.begin[k];
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    const f64x2 *part = (const f64x2 *)ws.partials + first;
    a0 = 0.0;
    a1 = 0.0;
    constexpr int U = DEDLOC_TRUST_UNROLL;  // loads in flight per lane
    for (uint32_t i0 = 0; i0 < ntiles; i0 += U * kWG) {
        f64x2 q[U];
#pragma unroll
        for (int j = 0; j < U; j++) {
            const uint32_t i = i0 + j * kWG + threadIdx.x;
            q[j] = i < ntiles ? part[i] : f64x2{0.0, 0.0};
        }
#pragma unroll
        for (int j = 0; j < U; j++) {
            a0 += q[j][0];
            a1 += q[j][1];
        }
    }
    block_sum2(a0, a1);
}

// The trust ratio of tensor k inside pass B.  One workgroup of the tensor,
// the producer (dispatched ahead of every other tile), sums the partials
// and publishes r in the tensor's workspace word as (epoch << 32 | bits of
// r) with one relaxed device-scope atomic store; the others poll that word
// with relaxed device-scope atomic loads until it carries this launch's
// epoch (a value and its tag in one word: no ordering between two
// locations is needed).  The epoch is a workspace counter that pass A
// advances on every launch plus a value the host draws for every call, so
// every call, graph replays included, has a tag that no word left by an
// earlier call on this workspace carries (and that other contents match
// only by a 2^-32 chance).  The polling is bounded: a workgroup that gives up
// sums the partials itself, in the same order, so r is the same bits on
// every path and every kernel exits.  Every thread calls it.
template <int OPT>
__device__ __forceinline__ float tensor_ratio(const Chunk &ch, const OptParams &op, const TileWs &ws,
                                              uint32_t k, bool producer, uint32_t epoch,
                                              float *__restrict__ trust_out) {
    __shared__ float s_r;
    __shared__ int s_have;
    unsigned long long *word = ws.trust + ch.t0 + k;
    if (!producer) {
        if (threadIdx.x == 0) {
            int have = 0;
            unsigned bits = 0u;
            for (uint32_t i = 0; i < op.trust_polls; i++) {
                const unsigned long long w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((uint32_t)(w >> 32) == epoch) {
                    have = 1;
                    bits = (uint32_t)w;
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
            }
            s_have = have;
            s_r = __uint_as_float(bits);
        }
        __syncthreads();
        if (s_have) return s_r;  // workgroup-uniform
    }
    double a0, a1;
    tensor_sums(ch, ws, k, a0, a1);
    if (threadIdx.x == 0) {
        const float r = trust_ratio<OPT>(ch.flags[k], op, a0, a1);
        if (producer) {
            __hip_atomic_store(word, ((unsigned long long)epoch << 32) | __float_as_uint(r), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            if (trust_out) trust_out[ch.t0 + k] = r;
        }
        s_r = r;
    }
    __syncthreads();
    return s_r;
}

// Pass B.  LAMB: x' = x - (lr * r_t) * u, with u recomputed from x, m', v' by
// the same operations as pass A.  LARS: v' = fma(mu, v, (lr*r_t)*(g + lambda*x)),
// x' = x - v', with g read again from the gathered message (SRC).  The
// tile's data are loaded and the step direction formed before r_t is known.
template <int SRC, int OPT, bool NT>
__global__ __launch_bounds__(kWG) void opt_b_kernel(const Chunk ch, const GradArgs ga, const OptParams op,
                                                    float *__restrict__ x, float *__restrict__ m,
                                                    float *__restrict__ v, TileWs ws, uint32_t nonce,
                                                    float *__restrict__ trust_out) {
    // Workgroups [0, nt) are the producers: tile 0 of tensor k = blockIdx.x
    // (the producer of an empty tensor writes r = 1 and exits).  The rest
    // cover every tile b of the chunk, last to first (the re-reads start with
    // what pass A touched last), and skip tile 0.
    uint32_t k, tile;
    const bool producer = blockIdx.x < ch.nt;
    if (producer) {
        k = blockIdx.x;
        tile = 0;
        if (ch.begin[k] == ch.begin[k + 1]) {
            if (threadIdx.x == 0 && trust_out) trust_out[ch.t0 + k] = 1.0f;
            return;
        }
    } else {
        const uint32_t b = gridDim.x - 1 - blockIdx.x;
        k = chunk_tensor(ch, b);
        tile = b - ch.begin[k];
        if (tile == 0) return;
    }
    const uint64_t t_hi = ch.base + ch.start[k + 1];
    const float lam = (ch.flags[k] & 1u) ? op.wd : 0.0f;
    const uint32_t epoch = ws.epoch[0] + nonce;  // ws.epoch: advanced by this chunk's pass A
    // the producer publishes r_t before touching its own tile (its partial
    // loads would otherwise queue behind the tile's loads)
    float lrr = producer ? op.lr * tensor_ratio<OPT>(ch, op, ws, k, true, epoch, trust_out) : 0.0f;
    const uint64_t e0 = ch.base + ch.start[k] + (uint64_t)tile * kRow + threadIdx.x * kVec;
    const int cnt = count8(e0, t_hi);
    float xv[8], dv[8], vv[8];
    if (cnt > 0) {
        load8<NT>(x, e0, cnt, xv);
        load8<NT>(v, e0, cnt, vv);
        if (OPT == kOptLamb) {
            float mv[8];
            load8<NT>(m, e0, cnt, mv);
#pragma unroll
            for (int j = 0; j < 8; j++) dv[j] = lamb_dir(mv[j], vv[j], xv[j], lam, op);
        } else {
            float g[8];
            load_grad<SRC, kPeerBatch, true>(ga, PeerTable{}, e0, cnt, g);
#pragma unroll
            for (int j = 0; j < 8; j++) dv[j] = g[j] + lam * xv[j];
        }
    }
    if (!producer) lrr = op.lr * tensor_ratio<OPT>(ch, op, ws, k, false, epoch, trust_out);
    if (cnt > 0) {
        if (OPT == kOptLamb) {
#pragma unroll
            for (int j = 0; j < 8; j++) xv[j] = xv[j] - lrr * dv[j];
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++) {
                vv[j] = fmaf(op.momentum, vv[j], lrr * dv[j]);
                xv[j] = xv[j] - vv[j];
            }
            store8<NT>(v, e0, cnt, vv);
        }
        store8<NT>(x, e0, cnt, xv);
    }
}

// ------------------------------------------------------ LAMB in one pass

// A row of LAMB's one pass, without gaps in a wave's accesses (GF: row_at's
// layout).  The fused average keeps eight consecutive elements per lane, which
// its 16-byte message accesses need.
template <bool GF>
struct Row {
    uint64_t row, t_hi;
    __device__ __forceinline__ Row(uint64_t row_, uint64_t t_hi_) : row(row_), t_hi(t_hi_) {}
    __device__ __forceinline__ bool full() const { return row + kRow <= t_hi; }  // workgroup-uniform
    __device__ __forceinline__ uint64_t e0() const { return row + threadIdx.x * kVec; }
    // whether the lane's element j (0..7) lies in the tensor
    __device__ __forceinline__ bool has(int j) const {
        return GF ? row + row_at(j >> 2) + (j & 3) < t_hi : e0() + j < t_hi;
    }
    // the lane's eight elements (zero past the end)
    template <bool NT = true>
    __device__ __forceinline__ void load(const float *__restrict__ p, float *o) const {
        if (!GF) {
            load8<NT>(p, e0(), count8(e0(), t_hi), o);
        } else if (full()) {
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const f32x4 *q = (const f32x4 *)(p + row + row_at(h));
                const f32x4 a = NT ? __builtin_nontemporal_load(q) : *q;
#pragma unroll
                for (int j = 0; j < 4; j++) o[4 * h + j] = a[j];
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++) o[j] = has(j) ? p[row + row_at(j >> 2) + (j & 3)] : 0.0f;
        }
    }
    __device__ __forceinline__ void store(float *__restrict__ p, const float *o) const {
        if (!GF) {
            store8<true>(p, e0(), count8(e0(), t_hi), o);
        } else if (full()) {
#pragma unroll
            for (int h = 0; h < 2; h++)
                __builtin_nontemporal_store(f32x4{o[4 * h], o[4 * h + 1], o[4 * h + 2], o[4 * h + 3]},
                                            (f32x4 *)(p + row + row_at(h)));
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++)
                if (has(j)) p[row + row_at(j >> 2) + (j & 3)] = o[j];
        }
    }
};

// The gradient of a row from a message (or an fp32 gradient) as loaded, so
// that the loads can be in flight while another row is worked on.
template <int SRC>
struct RawGrad {
    float g[SRC == kSrcF32 ? 8 : 1];
    u32x4 c;     // fp16: the lane's eight codes; int8: two words of four
    float s[2];  // int8: the block scales of the two words
    __device__ __forceinline__ void load(const GradArgs &ga, const Row<true> &r) {
        const uint64_t row = r.row;
        if (SRC == kSrcF32) {
            r.load((const float *)ga.grad, g);
        } else if (SRC == kSrcFP16) {
            const uint16_t *p = (const uint16_t *)ga.grad;
            if (r.full()) {
                const u32x2 a = ld_stream((const u32x2 *)(p + row + row_at(0)));
                const u32x2 b = ld_stream((const u32x2 *)(p + row + row_at(1)));
                c = u32x4{a[0], a[1], b[0], b[1]};
            } else {
                c = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < 8; j++)
                    if (r.has(j)) c[j >> 1] |= (unsigned)p[row + row_at(j >> 2) + (j & 3)] << (16 * (j & 1));
            }
        } else if (SRC == kSrcI8) {
            const int8_t *p = (const int8_t *)ga.grad;
#pragma unroll
            for (int h = 0; h < 2; h++) {  // rows start at multiples of 8: four codes share a block
                const uint64_t e = row + row_at(h);
                if (r.full()) {
                    c[h] = ld_stream((const unsigned *)(p + e));
                    s[h] = ga.scales[e / kI8Block];
                } else {
                    c[h] = 0u;
                    s[h] = e < r.t_hi ? ga.scales[e / kI8Block] : 0.0f;
#pragma unroll
                    for (int j = 0; j < 4; j++)
                        if (e + j < r.t_hi) c[h] |= (unsigned)(uint8_t)p[e + j] << (8 * j);
                }
            }
        }
    }
    __device__ __forceinline__ void decode(float *o) const {
        if (SRC == kSrcF32) {
#pragma unroll
            for (int j = 0; j < 8; j++) o[j] = g[j];
        } else if (SRC == kSrcFP16) {
            unpack_fp16x8(c, o);
        } else if (SRC == kSrcI8) {
#pragma unroll
            for (int j = 0; j < 8; j++) o[j] = sbyte(c[j >> 2], j & 3) * s[j >> 2];
        }
    }
};

// Partial sums (x^2 and u^2) as four words, each half of a double under the
// call's tag: whoever reads a word sees from it alone whether this launch
// wrote it, so no ordering between two locations (a release fence: on gfx950
// a full L2 write-back) is needed.
__device__ __forceinline__ void put_part(unsigned long long *w, uint32_t tag, double a, double b) {
    const unsigned long long t = (unsigned long long)tag << 32;
    const unsigned long long ab = (unsigned long long)__double_as_longlong(a);
    const unsigned long long bb = (unsigned long long)__double_as_longlong(b);
    __hip_atomic_store(w, t | (ab & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 1, t | (ab >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 2, t | (bb & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 3, t | (bb >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The sums of a record, and whether all four words carry the tag.
__device__ __forceinline__ bool get_part(const unsigned long long *w, uint32_t tag, double &a, double &b) {
    unsigned long long q[4];
#pragma unroll
    for (int i = 0; i < 4; i++) q[i] = __hip_atomic_load(w + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    a = __longlong_as_double((long long)((q[1] << 32) | (q[0] & 0xffffffffull)));
    b = __longlong_as_double((long long)((q[3] << 32) | (q[2] & 0xffffffffull)));
    return (uint32_t)(q[0] >> 32) == tag && (uint32_t)(q[1] >> 32) == tag && (uint32_t)(q[2] >> 32) == tag &&
           (uint32_t)(q[3] >> 32) == tag;
}

// Whether a wait ends with poll i.  Once every workgroup of the grid runs,
// whatever is waited for comes, and waiting for the slower ones is where the
// faster ones belong (up to 400 polls in a round of 64 peers, more on 500M
// elements).  While other work on the GPU keeps some of them from starting, a
// wait may be for them, so it ends after 48 polls (some 40 us) and the tensor is
// left to pass B; after that no wait of the launch is longer than 16.
// Workgroups are dispatched in order on each of the (at most 8) XCDs, so with
// the grid's last 8 running all are.  (Two steps of 2^25 elements in one tensor
// on two streams, each keeping part of the other's grid from starting: 541 us the
// pair with a bound of 512 polls, 460 with this, 437 one after the other.)
__device__ __forceinline__ bool stop_waiting(const LineWs &ws, uint32_t tag, uint32_t i) {
    if (i % 16 != 15) return false;
    const unsigned long long w = __hip_atomic_load(ws.state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (uint32_t)w == tag || (i + 1 >= kLineShortWait && (uint32_t)(w >> 32) != kLineLast);
}

// The sums of a record once it is there, polling at most `polls` times, and less
// once any tensor of the launch was given up.
__device__ __forceinline__ bool wait_part(const LineWs &ws, const unsigned long long *w, uint32_t tag, uint32_t polls,
                                          double &a, double &b) {
    for (uint32_t i = 0; i < polls; i++) {
        if (get_part(w, tag, a, b)) return true;
        if (stop_waiting(ws, tag, i)) break;
        __builtin_amdgcn_s_sleep(4);
    }
    return false;
}

// Sums over a tensor of its records [0, n) from `part` on without number
// `own`, by the whole workgroup, in a fixed order: thread-strided, then a
// fixed tree.  At most three records a thread, since each workgroup of the grid
// (three per CU) leaves one per tensor.  WAIT: poll for records not yet written
// (bounded); otherwise all of them are there.  Returns whether every record was
// seen; thread 0 gets the sums.
template <bool WAIT>
__device__ __forceinline__ bool record_sums(const LineWs &ws, const unsigned long long *part, uint32_t n, uint32_t own,
                                            uint32_t tag, uint32_t polls, double &a0, double &a1) {
    bool ok = true;
    a0 = 0.0;
    a1 = 0.0;
    for (uint32_t i = threadIdx.x; i < n && ok; i += kWG) {
        double p = 0.0, q = 0.0;
        if (i != own) {
            if (WAIT) ok = wait_part(ws, part + 4 * (uint64_t)i, tag, polls, p, q);
            else get_part(part + 4 * (uint64_t)i, tag, p, q);
        }
        a0 += p;
        a1 += q;
    }
    const bool all = !WAIT || __syncthreads_and(ok);
    block_sum2(a0, a1);
    return all;
}

// Unit b of the chunk: two rows of one tensor (the tensor's last unit may
// have one, and end within a row).
struct UnitAt {
    uint32_t k, unit, units;
    uint64_t row, t_hi;  // first element, end of the tensor
    // hint: a tensor that may well be it
    __device__ __forceinline__ UnitAt(const Chunk &ch, uint32_t b, uint32_t hint) {
        k = ch.begin[hint] <= b && b < ch.begin[hint + 1] ? hint : chunk_tensor(ch, b);
        unit = b - ch.begin[k];
        units = ch.begin[k + 1] - ch.begin[k];
        row = ch.base + ch.start[k] + (uint64_t)unit * (2 * kRow);
        t_hi = ch.base + ch.start[k + 1];
    }
    // Kept on chip until its tensor's ratio is known.
    __device__ __forceinline__ bool held(const OptParams &op) const { return units - 1 - unit < op.hold; }
};

// The records of tensor k, in its 16 bytes of workspace per row (32 per unit,
// of which the last may have 16): one record of 32 bytes for each workgroup
// that has units of it (record_of).  The workgroup of the last unit forms the
// ratio and leaves its two sums untagged (pass B reads them after the launch).
// A record per unit instead took the owner 2^e / 2^20 dependent reads on a
// tensor of 2^e elements: longer than the others wait (2^28 elements 34 ms
// instead of 1.9).
__device__ __forceinline__ unsigned long long *tensor_parts(const Chunk &ch, const LineWs &ws, uint32_t k) {
    return ws.part + 2 * (uint64_t)(ch.row_base + 2 * ch.begin[k] - ch.odd_before[k]);
}

// Number of a workgroup's record: its unit's where no workgroup has two units
// of the tensor, else its own (there are then more than G units, so number
// G - 1 has 32 bytes).
__device__ __forceinline__ uint32_t record_of(uint32_t unit, uint32_t units, uint32_t G, uint32_t group) {
    return units > G ? group : unit;
}

// The word of a tensor decides for all of it: (tag << 32) | bits of r once
// the ratio is known, or (tag << 32) | kFailed if a workgroup stopped waiting
// for it first; whichever is swapped in first stays.  Every wait is bounded,
// so every workgroup exits, whatever else runs on the GPU.
constexpr uint32_t kFailed = 0xffffffffu;  // no r: its only NaN is the canonical one

// Swap `low` in unless the word is decided already; returns what it holds.
__device__ __forceinline__ uint32_t decide(unsigned long long *word, unsigned long long seen, uint32_t tag, uint32_t low) {
    while ((uint32_t)(seen >> 32) != tag) {
        if (__hip_atomic_compare_exchange_strong(word, &seen, ((unsigned long long)tag << 32) | low, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            return low;
    }
    return (uint32_t)seen;
}

// Wait for the word's decision (`seen`: its content when last looked at).  A
// lane that only follows another on the same word (`mine` false) decides nothing
// and has no answer: a compare-and-swap by 64 lanes on one word takes 64 turns.
__device__ __forceinline__ uint32_t await_ratio(const LineWs &ws, uint32_t polls, unsigned long long *word,
                                                unsigned long long seen, uint32_t tag, bool mine) {
    for (uint32_t i = 0; i < polls && (uint32_t)(seen >> 32) != tag; i++) {
        if (stop_waiting(ws, tag, i)) break;
        __builtin_amdgcn_s_sleep(4);
        seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if ((uint32_t)(seen >> 32) == tag) return (uint32_t)seen;
    uint32_t got = kFailed;
    if (mine) {
        got = decide(word, seen, tag, kFailed);
        if (got == kFailed) __hip_atomic_store((uint32_t *)ws.state, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return got;
}

// LAMB in one pass: per row the gradient (optionally the fused average), the
// new moments, and the sums of x^2 and u^2.  x and u then wait on chip, in a
// line of NR register slots and NL LDS slots (rows) per workgroup, until the
// tensor's trust ratio is known, and x' = x - (lr*r_t)*u is written.  The grid
// is persistent: workgroup w takes units w, w + gridDim.x, ...
template <int SRC>
__global__ __launch_bounds__(kWG, kLineGroups) void lamb_a_kernel(const Chunk ch, const PeerTable pt,
                                                          const GradArgs ga, const OptParams op,
                                                          float *__restrict__ x,
                                                          float *__restrict__ m, float *__restrict__ v,
                                                          LineWs ws, uint32_t nonce, float *__restrict__ trust_out) {
    constexpr uint32_t NR = kLineRegs, NL = kLineLds, S = NR + NL;
    constexpr bool kPeers = SRC >= kSrcPeersFP16, GF = !kPeers;
    __shared__ f32x4 park[4 * NL][kWG];
    const uint32_t G = gridDim.x, n = ch.begin[ch.nt];
    const uint32_t epoch = ws.epoch[0];
    const uint32_t tag = epoch + nonce;
    // the tag as pass B reads it (ws.epoch[0] is advanced there, and read
    // here only)
    if (blockIdx.x == 0 && threadIdx.x == 0) ws.epoch[1] = epoch;
    // the grid's last workgroups say that they run (for a smaller grid's missing
    // ones workgroup 0 does)
    if (blockIdx.x + kLineLast >= G && threadIdx.x == 0)
        __hip_atomic_fetch_add((uint32_t *)ws.state + 1, blockIdx.x == 0 ? kLineLast - G + 1 : 1u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    float xr[NR][8], dr[NR][8];
    uint32_t slot = 0, it = 0;  // slot: (it - NR) % NL
    auto unpark = [&](uint32_t sl, float *xp, float *dp) {
#pragma unroll
        for (int q = 0; q < 2; q++) {
            const f32x4 a = park[4 * sl + q][threadIdx.x], d = park[4 * sl + 2 + q][threadIdx.x];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                xp[4 * q + j] = a[j];
                dp[4 * q + j] = d[j];
            }
        }
    };
    auto apply = [&](const Row<GF> &r, float lrr, const float *xp, const float *dp) {
        float xn[8];
#pragma unroll
        for (int j = 0; j < 8; j++) xn[j] = xp[j] - lrr * dp[j];
        r.store(x, xn);
    };
    float fx[8], fm[8], fv[8];  // the next row's state
    RawGrad<SRC> fg;
    auto fetch = [&](const Row<GF> &r) {
        if (r.row >= r.t_hi) return;
        // x plain, m and v and all stores non-temporal: a cache that still holds
        // part of x from the last call serves it (non-temporal / plain; the same
        // buffers again: 40M elements' round 380 / 370 us, the step on 60M 360 / 352,
        // ALBERT-large's round alone 191 / 187; three sets in turn: 400 / 390, 360 /
        // 352, ALBERT-xlarge's round 967 / 959, the step on 17.7M 98.8 / 97.4).  With
        // more of them plain the same buffers again gain more and others lose more:
        // ALBERT-large's round with all loads 186 / 221, all 184 / 224, m's loads and
        // stores 193 / 215.  Beside the local gradient, which is read plainly too,
        // only the same buffers gain: ALBERT-large 203 / 201, three sets 204.6 / 206.5
        // (with the gradient non-temporal instead 207 and 210).
        r.template load<SRC == kSrcPeersFP16Local>(x, fx);
        r.load(m, fm);
        r.load(v, fv);
        if constexpr (!kPeers) fg.load(ga, r);
        // a message's step waits here: with the loads left in flight over the
        // sums and the leaving row's stores it ran 101 instead of 98 us on
        // ALBERT-large (the fused average the other way round: 188 against 198)
        if (!kPeers) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    };
    UnitAt t(ch, blockIdx.x, 0), to(ch, blockIdx.x, 0);
    fetch(Row<GF>(t.row, t.t_hi));
    double s0 = 0.0, s1 = 0.0;
    uint32_t b = blockIdx.x;
#pragma unroll 1
    for (;; it++) {
        const uint32_t half = it & 1;
        const Row<GF> r(t.row + (uint64_t)half * kRow, t.t_hi);
        // the row that leaves the line in this turn: its tensor's word is
        // loaded while the new row is worked on
        if (it >= S && (it - S) % 2 == 0) to = UnitAt(ch, blockIdx.x + (it - S) / 2 * G, to.k);
        const Row<GF> ro(to.row + (uint64_t)((it - S) & 1) * kRow, to.t_hi);
        const bool leaves = it >= S && to.held(op) && ro.row < to.t_hi;
        unsigned long long q = 0;
        if (leaves) q = __hip_atomic_load(ws.trust + ch.t0 + to.k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        float xv[8], dv[8];
        if (kPeers ? r.e0() < r.t_hi : r.row < r.t_hi) {
            const float lam = (ch.flags[t.k] & 1u) ? op.wd : 0.0f;
            float g[8], mv[8], vv[8];
            if constexpr (kPeers) load_grad<SRC, kLinePeerBatch, false>(ga, pt, r.e0(), count8(r.e0(), r.t_hi), g);
            else fg.decode(g);
#pragma unroll
            for (int j = 0; j < 8; j++) {
                xv[j] = fx[j];
                mv[j] = fmaf(op.beta1, fm[j], op.omb1 * g[j]);
                vv[j] = fmaf(op.beta2, fv[j], op.omb2 * (g[j] * g[j]));
                dv[j] = lamb_dir(mv[j], vv[j], xv[j], lam, op);
                // past the end: no part of the sums, whatever eps and c2 are
                if (!r.full() && !r.has(j)) dv[j] = 0.0f;
                s0 += (double)xv[j] * (double)xv[j];
                s1 += (double)dv[j] * (double)dv[j];
            }
            r.store(m, mv);
            r.store(v, vv);
        }
        const bool more = half == 0 || b + G < n;
        const UnitAt tn = half == 0 || b + G >= n ? t : UnitAt(ch, b + G, t.k);
        if (more) fetch(half == 0 ? Row<GF>(r.row + kRow, r.t_hi) : Row<GF>(tn.row, tn.t_hi));
        if (half == 1 && t.unit + G >= t.units) {  // the workgroup's last unit of the tensor
            block_sum2(s0, s1);
            const uint32_t rec = record_of(t.unit, t.units, G, blockIdx.x);
            unsigned long long *part = tensor_parts(ch, ws, t.k);
            if (t.unit != t.units - 1) {
                if (threadIdx.x == 0) put_part(part + 4 * (uint64_t)rec, tag, s0, s1);
            } else {
                // the workgroup of the tensor's last unit publishes its ratio
                double a0 = 0.0, a1 = 0.0;
                const uint32_t n_rec = t.units < G ? t.units : G;
                const bool ok = n_rec == 1 || record_sums<true>(ws, part, n_rec, rec, tag, op.trust_polls, a0, a1);
                if (threadIdx.x == 0) {
                    double *own = (double *)(part + 4 * (uint64_t)rec);
                    own[0] = s0;
                    own[1] = s1;
                    unsigned long long *word = ws.trust + ch.t0 + t.k;
                    const float rt = trust_ratio<kOptLamb>(ch.flags[t.k], op, a0 + s0, a1 + s1);
                    const uint32_t low = ok ? __float_as_uint(rt) : kFailed;
                    const unsigned long long seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const uint32_t got = decide(word, seen, tag, low);
                    if (got == kFailed) __hip_atomic_store((uint32_t *)ws.state, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    else if (trust_out) trust_out[ch.t0 + t.k] = rt;
                }
            }
            s0 = s1 = 0.0;
        }
        if (leaves) {
            const uint32_t low = __builtin_amdgcn_readfirstlane(
                await_ratio(ws, op.trust_polls, ws.trust + ch.t0 + to.k, q, tag, (threadIdx.x & 63) == 0));
            if (low != kFailed) {
                float xp[8], dp[8];
                unpark(slot, xp, dp);
                apply(ro, op.lr * __uint_as_float(low), xp, dp);
            }
        }
        if (it >= NR) {
            const float *xo = xr[NR - 1], *d = dr[NR - 1];
#pragma unroll
            for (int c = 0; c < 2; c++) {
                park[4 * slot + c][threadIdx.x] = f32x4{xo[4 * c], xo[4 * c + 1], xo[4 * c + 2], xo[4 * c + 3]};
                park[4 * slot + 2 + c][threadIdx.x] = f32x4{d[4 * c], d[4 * c + 1], d[4 * c + 2], d[4 * c + 3]};
            }
            slot = slot + 1 == NL ? 0 : slot + 1;
        }
#pragma unroll
        for (uint32_t i = NR - 1; i > 0; i--)
#pragma unroll
            for (int j = 0; j < 8; j++) {
                xr[i][j] = xr[i - 1][j];
                dr[i][j] = dr[i - 1][j];
            }
#pragma unroll
        for (int j = 0; j < 8; j++) {
            xr[0][j] = xv[j];
            dr[0][j] = dv[j];
        }
        if (!more) break;
        t = tn;
        if (half == 1) b += G;
    }
    it++;
    // the rows still in the line: the one taken i turns before the end (`it`
    // turns in all) has slot i - 1
    const uint32_t left = it < S ? it : S;
    uint32_t r_lane = kFailed;
    if ((threadIdx.x & 63) < left) {
        const UnitAt u(ch, blockIdx.x + (it - 1 - (threadIdx.x & 63)) / 2 * G, t.k);
        unsigned long long *word = ws.trust + ch.t0 + u.k;
        if (u.held(op))
            r_lane = await_ratio(ws, op.trust_polls, word, __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), tag,
                                 true);
    }
    for (uint32_t i = left; i > 0; i--) {
        const UnitAt u(ch, blockIdx.x + (it - i) / 2 * G, t.k);
        const Row<GF> r(u.row + (uint64_t)((it - i) & 1) * kRow, u.t_hi);
        const uint32_t low = __builtin_amdgcn_readfirstlane(__shfl(r_lane, i - 1, 64));
        if (r.row >= r.t_hi || !u.held(op) || low == kFailed) continue;
        float xp[8], dp[8];
        if (i > NR) {
            // parked in turn: the newest parked row (i = NR + 1) is just before `slot`
            const uint32_t back = i - NR;
            unpark(slot >= back ? slot - back : slot + NL - back, xp, dp);
        } else {
#pragma unroll
            for (uint32_t c = 0; c < NR; c++)
                if (i == c + 1)
#pragma unroll
                    for (int j = 0; j < 8; j++) {
                        xp[j] = xr[c][j];
                        dp[j] = dr[c][j];
                    }
        }
        apply(r, op.lr * __uint_as_float(low), xp, dp);
    }
}

// A row from memory: u formed again by pass A's operations.
__device__ __forceinline__ void redo_row(const OptParams &op, float *__restrict__ x, float *__restrict__ m,
                                         float *__restrict__ v, uint64_t row, uint64_t t_hi, float lam, float lrr) {
    const Row<true> r(row, t_hi);
    float xv[8], mv[8], vv[8];
    r.load(x, xv);
    r.load(m, mv);
    r.load(v, vv);
#pragma unroll
    for (int j = 0; j < 8; j++) xv[j] = xv[j] - lrr * lamb_dir(mv[j], vv[j], xv[j], lam, op);
    r.store(x, xv);
}

// The ratio of tensor k, which pass A gave up, from its records; G: pass A's grid.
__device__ __forceinline__ float settled_ratio(const Chunk &ch, const OptParams &op, const LineWs &ws, uint32_t k,
                                               uint32_t G, uint32_t tag) {
    const uint32_t units = ch.begin[k + 1] - ch.begin[k];
    const uint32_t n_rec = units < G ? units : G, own_rec = record_of(units - 1, units, G, (ch.begin[k + 1] - 1) % G);
    const unsigned long long *part = tensor_parts(ch, ws, k);
    const double *own = (const double *)(part + 4 * (uint64_t)own_rec);
    __shared__ float s_r;
    double a0, a1;
    record_sums<false>(ws, part, n_rec, own_rec, tag, 0, a0, a1);
    if (threadIdx.x == 0) s_r = trust_ratio<kOptLamb>(ch.flags[k], op, a0 + own[0], a1 + own[1]);
    __syncthreads();
    return s_r;  // written again only past another barrier
}

// The ratio of tensor k, of which pass A left rows, for one of the workgroups
// of those rows: as pass A decided it; else the tensor's first workgroup
// (`first`, dispatched ahead of its others) settles it once and publishes it in
// the record after the last, which the others poll a bounded number of times
// before they settle it themselves, in the same order.  (Such a tensor has more
// than 2 * G units, so that record is within its workspace.)
__device__ __forceinline__ float rest_ratio(const Chunk &ch, const OptParams &op, const LineWs &ws, uint32_t k, bool first,
                                            uint32_t G, uint32_t tag) {
    const unsigned long long w = ws.trust[ch.t0 + k];
    if ((uint32_t)(w >> 32) == tag && (uint32_t)w != kFailed) return __uint_as_float((uint32_t)w);
    unsigned long long *late = tensor_parts(ch, ws, k) + 4 * (uint64_t)G;
    if (!first) {
        __shared__ unsigned long long s_late;
        if (threadIdx.x == 0) {
            unsigned long long seen = 0;
            for (uint32_t i = 0; i < op.trust_polls; i++) {
                seen = __hip_atomic_load(late, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((uint32_t)(seen >> 32) == tag) break;
                __builtin_amdgcn_s_sleep(4);
            }
            s_late = seen;
        }
        __syncthreads();
        if ((uint32_t)(s_late >> 32) == tag && op.trust_polls > 0) return __uint_as_float((uint32_t)s_late);
    }
    const float r = settled_ratio(ch, op, ws, k, G, tag);
    if (first && threadIdx.x == 0)
        __hip_atomic_store(late, ((unsigned long long)tag << 32) | __float_as_uint(r), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    return r;
}

// What pass A left: the rows of units it does not hold (workgroups
// [0, n_rest), last to first: the re-reads start with what pass A touched
// last), and all held rows of tensors that were given up, if there are any.
// Also r = 1 of empty tensors, and the next launch's tag and state.
__global__ __launch_bounds__(kWG) void lamb_b_kernel(const Chunk ch, const RestTable rt, const OptParams op,
                                                     float *__restrict__ x, float *__restrict__ m,
                                                     float *__restrict__ v, LineWs ws, uint32_t nonce,
                                                     float *__restrict__ trust_out) {
    const uint32_t epoch = ws.epoch[1];
    const uint32_t tag = epoch + nonce;
    if (blockIdx.x < rt.n_rest) {
        const uint32_t q = rt.n_rest - 1 - blockIdx.x;
        uint32_t lo = 0, hi = ch.nt;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (rt.begin[mid] <= q) lo = mid;
            else hi = mid;
        }
        const uint64_t row = ch.base + ch.start[lo] + (uint64_t)(q - rt.begin[lo]) * kRow;
        const float lam = (ch.flags[lo] & 1u) ? op.wd : 0.0f;
        const float lrr = op.lr * rest_ratio(ch, op, ws, lo, q + 1 == rt.begin[lo + 1], rt.grid_a, tag);
        redo_row(op, x, m, v, row, ch.base + ch.start[lo + 1], lam, lrr);
        return;
    }
    const uint32_t q = blockIdx.x - rt.n_rest, step = gridDim.x - rt.n_rest;
    if (q == 0) {
        for (uint32_t k = threadIdx.x; k < ch.nt; k += kWG)
            if (trust_out && ch.begin[k] == ch.begin[k + 1]) trust_out[ch.t0 + k] = 1.0f;
        // (a chunk of empty tensors has no pass A, which alone sets epoch[1])
        if (threadIdx.x == 0 && ch.begin[ch.nt] > 0) {
            ws.epoch[0] = epoch + 1u;
            ((uint32_t *)ws.state)[1] = 0u;
        }
    }
    if (*(const uint32_t *)ws.state != tag) return;
    // The held rows of the tensors given up, one after the other, in equal
    // shares: a workgroup settles the ratios of the few tensors in its own.
    __shared__ uint32_t s_rows[kChunkTensors];
    for (uint32_t k = threadIdx.x; k < ch.nt; k += kWG) {
        const uint32_t units = ch.begin[k + 1] - ch.begin[k];
        const bool gone = units > 0 && ws.trust[ch.t0 + k] == (((unsigned long long)tag << 32) | kFailed);
        s_rows[k] = gone ? 2 * (units < op.hold ? units : op.hold) : 0;
    }
    __syncthreads();
    uint64_t all = 0;
    for (uint32_t k = 0; k < ch.nt; k++) all += s_rows[k];
    const uint64_t lo = all * q / step, hi = all * (q + 1) / step;
    uint64_t at = 0;  // rows of the tensors before k
    for (uint32_t k = 0; k < ch.nt && at < hi; at += s_rows[k], k++) {
        const uint64_t a = lo > at ? lo - at : 0, b = hi - at < s_rows[k] ? hi - at : s_rows[k];
        if (a >= b) continue;
        const uint64_t t_hi = ch.base + ch.start[k + 1];
        const float lam = (ch.flags[k] & 1u) ? op.wd : 0.0f;
        const float r_t = settled_ratio(ch, op, ws, k, rt.grid_a, tag);
        if (a == 0 && threadIdx.x == 0 && trust_out) trust_out[ch.t0 + k] = r_t;
        const uint32_t first = 2 * (ch.begin[k + 1] - ch.begin[k]) - s_rows[k];  // the first held row
        for (uint64_t i = first + a; i < first + b; i++) {
            const uint64_t row = ch.base + ch.start[k] + i * kRow;
            if (row < t_hi) redo_row(op, x, m, v, row, t_hi, lam, op.lr * r_t);
        }
    }
}

// ------------------------------------------------ local accumulation
// acc = fma(b, g, acc): a micro-batch of b samples with mean gradient g.
// acc is read again by the next micro-batch (plain accesses: the Infinity
// Cache keeps a vector of ordinary size), the gradient is not.
template <bool G16>
__global__ __launch_bounds__(kWG) void accumulate_kernel(float *__restrict__ acc, const void *__restrict__ grad,
                                                         uint64_t n, float b) {
    const uint64_t row = (uint64_t)blockIdx.x * kRow;
    if (row + kRow <= n) {
        f32x4 a[2], g[2];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            a[h] = *(const f32x4 *)(acc + row + row_at(h));
            if (G16) {
                const u32x2 c = ld_stream((const u32x2 *)((const uint16_t *)grad + row + row_at(h)));
                g[h] = f32x4{h2f(c[0] & 0xffffu), h2f(c[0] >> 16), h2f(c[1] & 0xffffu), h2f(c[1] >> 16)};
            } else {
                g[h] = ld_stream((const f32x4 *)((const float *)grad + row + row_at(h)));
            }
        }
#pragma unroll
        for (int h = 0; h < 2; h++) {
#pragma unroll
            for (int j = 0; j < 4; j++) a[h][j] = fmaf(b, g[h][j], a[h][j]);
            *(f32x4 *)(acc + row + row_at(h)) = a[h];
        }
    } else {
        for (uint64_t e = row + threadIdx.x; e < n; e += kWG)
            acc[e] = fmaf(b, G16 ? h2f(((const uint16_t *)grad)[e]) : ((const float *)grad)[e], acc[e]);
    }
}

// mean = acc / count, encoded fp16; acc zeroed when reset.
__global__ __launch_bounds__(kWG) void finalize_fp16_kernel(float *__restrict__ acc, uint64_t n, float count,
                                                            uint16_t *__restrict__ codes, int reset) {
    const uint64_t row = (uint64_t)blockIdx.x * kRow;
    if (row + kRow <= n) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            f32x4 *p = (f32x4 *)(acc + row + row_at(h));
            const f32x4 a = *p;
            st_msg((u32x2 *)(codes + row + row_at(h)), u32x2{f2h(a[0] / count) | (f2h(a[1] / count) << 16),
                                                             f2h(a[2] / count) | (f2h(a[3] / count) << 16)});
            if (reset) *p = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    } else {
        for (uint64_t e = row + threadIdx.x; e < n; e += kWG) {
            codes[e] = (uint16_t)f2h(acc[e] / count);
            if (reset) acc[e] = 0.0f;
        }
    }
}

// int8: one wave per 1024-element block, 16 elements per lane.
__global__ __launch_bounds__(kWG) void finalize_i8_kernel(float *__restrict__ acc, uint64_t n, float count,
                                                          int8_t *__restrict__ codes, float *__restrict__ scales,
                                                          int reset) {
    const uint64_t blk = (uint64_t)blockIdx.x * (kWG / 64) + (threadIdx.x >> 6);
    if (blk * kI8Block >= n) return;  // whole wave past the end
    float val[kI8PerLane];
    load_i8_lane(acc, n, blk, val);
#pragma unroll
    for (int j = 0; j < kI8PerLane; j++) val[j] = val[j] / count;
    float s;
    const u32x4 c = encode_i8_wave(val, s);
    store_i8_lane(codes, scales, n, blk, c, s);
    if (reset) {
        const uint64_t b0 = i8_lane_base(blk);
        if ((blk + 1) * kI8Block <= n) {
#pragma unroll
            for (int q = 0; q < 4; q++) *(f32x4 *)(acc + I8_ELEM(b0, q, 0)) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        } else {
#pragma unroll
            for (int q = 0; q < 4; q++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const uint64_t e = I8_ELEM(b0, q, r);
                    if (e < n) acc[e] = 0.0f;
                }
        }
    }
}

__global__ __launch_bounds__(kWG) void fill_zero_kernel(uint32_t *p, uint64_t n_words) {
    const uint64_t i = (uint64_t)blockIdx.x * kWG + threadIdx.x;
    if (i < n_words) p[i] = 0u;
}

// --------------------------------------------------------------- launchers

static inline unsigned grid_for(uint64_t items, uint64_t per_block) {
    return (unsigned)((items + per_block - 1) / per_block);
}

// Launch through hipLaunchKernel, whose return value is this launch's own
// status (hipGetLastError after a <<<>>> launch would also report an error
// left pending by an earlier, unrelated call of the caller's).  The
// arguments are converted to the kernel's parameter types and held while
// the runtime copies them into the kernel arguments.
template <typename K, typename Held, size_t... I>
static hipError_t launch_held(K kernel, dim3 grid, hipStream_t s, Held &held, std::index_sequence<I...>) {
    void *argv[] = {(void *)&std::get<I>(held)...};
    return hipLaunchKernel((const void *)kernel, grid, dim3(kWG), argv, 0, s);
}

template <typename... KArgs, typename... Args>
static hipError_t launch_kernel(void (*kernel)(KArgs...), dim3 grid, hipStream_t s, Args &&...args) {
    if (grid.x == 0 || grid.y == 0) return hipSuccess;  // nothing to do
    std::tuple<KArgs...> held(std::forward<Args>(args)...);
    return launch_held(kernel, grid, s, held, std::index_sequence_for<KArgs...>{});
}

#define DEDLOC_LAUNCH(grid, kernel, s, ...) return launch_kernel((kernel), (grid), (s), __VA_ARGS__)

hipError_t launch_encode_fp16(const float *x, uint64_t n, uint16_t *codes, hipStream_t s) {
    DEDLOC_LAUNCH(dim3(grid_for(n, (uint64_t)kWG * kVec)), encode_fp16_kernel, s, x, n, codes);
}

hipError_t launch_decode_fp16(const uint16_t *codes, uint64_t n, float *out, hipStream_t s) {
    const dim3 grid(grid_for(n, (uint64_t)kWG * kVec));
    if (n >= kNtDecodeFp16) DEDLOC_LAUNCH(grid, decode_fp16_kernel<true>, s, codes, n, out);
    DEDLOC_LAUNCH(grid, decode_fp16_kernel<false>, s, codes, n, out);
}

hipError_t launch_encode_i8(const float *x, uint64_t n, int8_t *codes, float *scales, hipStream_t s) {
    DEDLOC_LAUNCH(dim3(grid_for(n, (uint64_t)kI8Block * (kWG / 64))), encode_i8_kernel, s, x, n, codes, scales);
}

hipError_t launch_decode_i8(const int8_t *codes, const float *scales, uint64_t n, float *out,
                            hipStream_t s) {
    const dim3 grid(grid_for(n, (uint64_t)kI8Block * (kWG / 64)));
    if (n >= kNtDecodeI8) DEDLOC_LAUNCH(grid, decode_i8_kernel<true>, s, codes, scales, n, out);
    DEDLOC_LAUNCH(grid, decode_i8_kernel<false>, s, codes, scales, n, out);
}

// Groups of at most this many members take the small peer batch.
constexpr uint32_t kSmallGroup = 4;

static uint32_t largest_group(const GroupTable &gt) {
    uint32_t m = 0;
    for (uint32_t g = 0; g < gt.n_groups; g++) m = std::max(m, gt.gbegin[g + 1] - gt.gbegin[g]);
    return m;
}

hipError_t launch_reduce_fp16(const GroupTable &gt, uint64_t len, const ChainArgs &ca, hipStream_t s) {
    const dim3 grid(grid_for(len, (uint64_t)kWG * kVec), gt.n_groups);
    if (ca.local.pos < 0 && largest_group(gt) <= kSmallGroup)
        DEDLOC_LAUNCH(grid, reduce_fp16_kernel<(int)kSmallGroup>, s, gt, len, ca);
    DEDLOC_LAUNCH(grid, reduce_fp16_kernel<kPeerBatch>, s, gt, len, ca);
}

hipError_t launch_reduce_i8(const GroupTable &gt, uint64_t len, const ChainArgs &ca, uint32_t cus, hipStream_t s) {
    const dim3 grid(grid_for(len, (uint64_t)kI8Block * (kWG / 64)), gt.n_groups);
    // Few waves (under 16 a CU, 4 workgroups) and many peers: the serial chain of
    // batches is what the launch takes, so the loads go out 16 at a time (30 peers
    // on 256 CUs: 1M elements 31.9 us a round against 37.0, 3M 48.7 / 50.7; 6M the
    // other way round 77.7 / 73.1).  Also where batches of 4, of which 8 workgroups
    // a CU run at once, leave a second generation nearly empty (10.5M elements
    // 120.7 us against 125.7; 13M 169.3 / 168.0, 8M 88.8 / 84.1).
    const uint64_t groups = (uint64_t)grid.x * grid.y, at_once = 8ull * cus;
    if (largest_group(gt) > 12 && (groups < at_once / 2 || (groups > at_once && groups <= at_once * 3 / 2)))
        DEDLOC_LAUNCH(grid, reduce_i8_kernel<kI8FewWaves>, s, gt, len, ca);
    DEDLOC_LAUNCH(grid, reduce_i8_kernel<kI8Batch>, s, gt, len, ca);
}

hipError_t launch_lamb_a(int src, const Chunk &ch, uint32_t n_groups, const PeerTable &pt, const GradArgs &ga,
                         const OptParams &op, float *x, float *m, float *v, const LineWs &ws, uint32_t nonce,
                         float *trust_out, hipStream_t s) {
    const dim3 g(n_groups);
    switch (src) {
#define DEDLOC_CASE(SRC) \
    case SRC: DEDLOC_LAUNCH(g, lamb_a_kernel<SRC>, s, ch, pt, ga, op, x, m, v, ws, nonce, trust_out)
    DEDLOC_CASE(kSrcF32);
    DEDLOC_CASE(kSrcFP16);
    DEDLOC_CASE(kSrcI8);
    DEDLOC_CASE(kSrcPeersFP16);
    DEDLOC_CASE(kSrcPeersFP16Chain);
    DEDLOC_CASE(kSrcPeersFP16Local);
#undef DEDLOC_CASE
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_lamb_b(const Chunk &ch, const RestTable &rt, uint32_t n_check, const OptParams &op, float *x, float *m,
                         float *v, const LineWs &ws, uint32_t nonce, float *trust_out, hipStream_t s) {
    DEDLOC_LAUNCH(dim3(rt.n_rest + n_check), lamb_b_kernel, s, ch, rt, op, x, m, v, ws, nonce, trust_out);
}

template <int OPT>
static hipError_t launch_a(int src, const Chunk &ch, const PeerTable &p, const GradArgs &ga, const OptParams &op,
                           float *x, float *m, float *v, const TileWs &ws, hipStream_t s) {
    const dim3 g(ch.begin[ch.nt]);
    switch (src) {
#define DEDLOC_CASE(SRC) \
    case SRC: DEDLOC_LAUNCH(g, (opt_a_kernel<SRC, OPT>), s, ch, p, ga, op, x, m, v, ws)
    DEDLOC_CASE(kSrcF32);
    DEDLOC_CASE(kSrcFP16);
    DEDLOC_CASE(kSrcI8);
    DEDLOC_CASE(kSrcPeersFP16);
    DEDLOC_CASE(kSrcPeersFP16Chain);
    DEDLOC_CASE(kSrcPeersFP16Local);
#undef DEDLOC_CASE
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_opt_a(int opt, int src, const Chunk &ch, const PeerTable &p, const GradArgs &ga, const OptParams &op,
                        float *x, float *m, float *v, const TileWs &ws, hipStream_t s) {
    return opt == kOptLamb ? launch_a<kOptLamb>(src, ch, p, ga, op, x, m, v, ws, s)
                           : launch_a<kOptLars>(src, ch, p, ga, op, x, m, v, ws, s);
}

template <bool NT>
static hipError_t launch_lars_b(int src, dim3 g, const Chunk &ch, const GradArgs &ga, const OptParams &op, float *x,
                                float *v, const TileWs &ws, uint32_t nonce, float *trust_out, hipStream_t s) {
    float *m = nullptr;
    switch (src) {
    case kSrcF32: DEDLOC_LAUNCH(g, (opt_b_kernel<kSrcF32, kOptLars, NT>), s, ch, ga, op, x, m, v, ws, nonce, trust_out);
    case kSrcFP16: DEDLOC_LAUNCH(g, (opt_b_kernel<kSrcFP16, kOptLars, NT>), s, ch, ga, op, x, m, v, ws, nonce, trust_out);
    case kSrcI8: DEDLOC_LAUNCH(g, (opt_b_kernel<kSrcI8, kOptLars, NT>), s, ch, ga, op, x, m, v, ws, nonce, trust_out);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_opt_b(int opt, int src, bool nt, const Chunk &ch, const GradArgs &ga, const OptParams &op, float *x,
                        float *m, float *v, const TileWs &ws, uint32_t nonce, float *trust_out, hipStream_t s) {
    const dim3 g(ch.nt + ch.begin[ch.nt]);  // one producer per tensor, then every tile
    if (opt == kOptLamb)
        DEDLOC_LAUNCH(g, (opt_b_kernel<kSrcF32, kOptLamb, false>), s, ch, ga, op, x, m, v, ws, nonce, trust_out);
    return nt ? launch_lars_b<true>(src, g, ch, ga, op, x, v, ws, nonce, trust_out, s)
              : launch_lars_b<false>(src, g, ch, ga, op, x, v, ws, nonce, trust_out, s);
}

hipError_t launch_accumulate(float *acc, const void *grad, bool fp16, uint64_t n, float b, hipStream_t s) {
    if (fp16) DEDLOC_LAUNCH(dim3(grid_for(n, (uint64_t)kWG * kVec)), accumulate_kernel<true>, s, acc, grad, n, b);
    DEDLOC_LAUNCH(dim3(grid_for(n, (uint64_t)kWG * kVec)), accumulate_kernel<false>, s, acc, grad, n, b);
}

hipError_t launch_finalize_fp16(float *acc, uint64_t n, float count, uint16_t *codes, int reset, hipStream_t s) {
    DEDLOC_LAUNCH(dim3(grid_for(n, (uint64_t)kWG * kVec)), finalize_fp16_kernel, s, acc, n, count, codes, reset);
}

hipError_t launch_finalize_i8(float *acc, uint64_t n, float count, int8_t *codes, float *scales, int reset,
                              hipStream_t s) {
    DEDLOC_LAUNCH(dim3(grid_for(n, (uint64_t)kI8Block * (kWG / 64))), finalize_i8_kernel, s, acc, n, count, codes,
                  scales, reset);
}

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s) {
    const uint64_t words = bytes / 4;
    if (words == 0) return hipSuccess;
    DEDLOC_LAUNCH(dim3(grid_for(words, kWG)), fill_zero_kernel, s, (uint32_t *)p, words);
}

}  // namespace dedloc

// libnetkv -- NetKV decode-instance selection for MI355X (gfx950).
//
// Host runtime and HIP kernels behind the C ABI declared in include/netkv.h.
// Method: "NetKV: Network-Aware Decode Instance Selection for Disaggregated
// LLM Inference", Algorithm 1 with Eqs. (2)-(7), evaluated for a whole batch
// of requests against one telemetry snapshot.
//
// Data layout in device memory (all owned by the handle):
//   * holder index of the resident block hashes of all decodes: every
//     distinct resident hash once in a two-choice bucketized cuckoo set
//     (two 8-byte slots per bucket, 0 = empty; hash value 0 is reserved),
//     with a 32-bit holder value per slot -- one decode, or a row of a
//     holder bitmap pool (one bit per decode).  One lookup answers a
//     membership test for every decode at once.
//   * snapshot: tier_map u8[P*D], util f32[P*D] (row-major by prefill),
//     n_inflight u16[4*P] (tier-major), free_mem u64[D], queue u32[D],
//     batch u32[D], plus the admitted bytes of the previous batch u64[D];
//     derived per call: (seconds per token, constant part) float2 rows per
//     prefill, and per decode the load term and feasibility limit.
//
// A selection (netkv_select_batch) takes one of three forms with the same
// results (direct_batch and bounded_batch say which):
//   direct (small batches):
//     direct_kernel    -- everything in one launch, a wavefront or four per
//                         request (after derive_kernel with staged routes).
//   bounded (snapshots whose costs tell groups of 64 decodes apart, as
//   spread_kernel measures at the load calls):
//     derive_bound_kernel -- the cost factors, and bounds per (prefill, group).
//     match_kernel     -- holder values of every request's leading held blocks.
//     bounded_kernel   -- scores the groups that the bounds leave; top-k.
//   along the batch order (large batches of long runs or in small pools,
//   per-pair outputs, pools of more than 4,096 decodes), in launch order (a
//   batch of 2^16 requests or more runs derive_kernel, then
//   lead_holder_kernel and lead_kernel, on a second stream beside the others):
//   derive_kernel      -- per-call cost factors (Eqs. (3)-(7) split by what
//                         they depend on).
//   prep_kernel        -- validate requests, build hash-order keys.
//   sort kernels       -- stable radix sort into hash order (rocPRIM's for
//                         small and very large batches).
//   order_kernel       -- common leading run with the previous position,
//                         leaders (positions whose next block some decode
//                         holds), segmented-scan elements within each tile
//                         of positions, records.
//   tile_prefix_kernel -- the tiles' exclusive prefixes (the scan's second
//                         level).
//   lead_holder_kernel -- holder values of every leader's blocks.
//   sort kernels       -- stable sort into prefill order, writing the
//                         scoring records (or rocPRIM's sort and
//                         assemble_kernel).
//   lead_kernel        -- prefix lengths of every leader on every decode.
//   score_kernel       -- per pair: prefix length min(leader's, L*),
//                         feasibility and cost (Eqs. (2)-(7)), then the
//                         group's top-k; one wavefront per (run of requests,
//                         group of 64*C decodes); optional per-pair outputs.
//   reduce_kernel      -- merges the groups' keys into each request's top-k
//                         (not launched when one group covers the pool).
// Other calls:
//   derive_scen_kernel, sweep_kernel -- re-scoring under congestion
//                         scenarios from the leader rows; lanes over requests.
//   tier_inv_kernel    -- Proposition 2's tier-ranking inversion counts.
//   sequential kernels -- Algorithm 1's per-request in-flight increments,
//                         one workgroup per prefill instance, from the
//                         leader rows (small batches: direct_kernel's rows).
//   selection_bytes_kernel -- the selections' transfer sizes (Eq. (2)).
//   load_snapshot_kernel, check_snapshot_kernel -- a snapshot's copy and checks.
//   pair / parts / dedupe / build kernels -- build the holder index; whole_*
//                         kernels where its blocks cannot hold the hashes.
//   commit kernels     -- between-batch counter / queue / memory update.
// The flow-level transfer simulation is in flowsim.hip.
#include <hip/hip_runtime.h>
#include <rocprim/device/device_radix_sort.hpp>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "netkv.h"
#include "netkv_internal.h"

namespace {

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr uint32_t kXcds = 8;   // accelerator complex dies of an MI355X, each with its own L2
constexpr int kBlock = kWave * kWavesPerBlock;
constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kGoldenInv = 0xF1DE83E19937733Dull;   // kGolden * kGoldenInv = 1 mod 2^64
constexpr uint64_t kMix64 = 0xBF58476D1CE4E5B9ull;
constexpr uint64_t kEmptyKey = ~0ull; // empty top-k entry (sorts last)
// bytes of the static scratch array of the no-allocation selection (per device)
constexpr uint64_t kScratchBytes = 64ull << 20;

enum : uint32_t {
    kErrRequest = 1u,    // request header inconsistent
    kErrObservation = 2u,   // congestion observation outside [0, 1) or NaN
    kErrSelection = 4u,  // selection index out of range
    kErrTableFull = 8u,  // insertion found no free slot
    kErrFlow = kErrFlowBit,           // flow simulation: invalid flow set
    kErrFlowStall = kErrFlowStallBit,   // flow simulation: an iteration bound was reached
};

// ------------------------------------------------------------------ device data

struct Snap {
    const uint8_t *tier_map;
    const float *util;
    const uint16_t *n_inflight;
    const uint64_t *free_mem;
    const uint32_t *queue;
    const uint32_t *batch;
    float bw[4];
    float lat[4];
    float t_a, t_b, alpha;
    uint32_t beta_max;
    uint64_t m_min;
    uint32_t bpt;
    uint32_t block_tokens;
    uint32_t P, D;
    uint32_t policy;         // 0: full NetKV, 1: no live congestion, 2: neither congestion nor in-flight
    // derived once per call by derive_kernel (Eqs. (3)-(7) factored by (p, d) and d)
    const float2 *sl;        // [P][slp] per (p, d): seconds per non-cached token, and the
                             // constant part L_tau + alpha (T_queue + T_decode)
    uint32_t slp;            // row pitch of sl in elements (an odd number of 128-byte lines)
    const float2 *sr;        // like sl, for the staged (two-hop) route; null without one
    const float *dbase;      // [D] alpha (T_queue + T_decode)
    const uint64_t *dxlim;   // [D] x = l - lambda is feasible iff x < dxlim
};

// The holder index of the resident block hashes K_d of all decodes: every
// distinct resident hash once, in a bucketized two-choice cuckoo set (two
// candidate buckets of two 8-byte slots; 0 = empty), and in a parallel array
// the 32-bit holder value of the key in the same slot:
//   kHeldOne | d -- the hash is resident on decode d alone;
//   row          -- it is resident on two or more decodes, the set bits of
//                   row `row` of the bitmap pool (bit d % 64 of word d / 64).
// A hash that is not in the set is resident nowhere (kNoHolder).  One lookup
// answers a membership test for every decode at once.
constexpr uint32_t kHeldOne = 0x80000000u;
constexpr uint32_t kNoHolder = 0xFFFFFFFFu;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

struct Table {
    const uint64_t *keys;   // [buckets][2] distinct resident hashes
    const uint32_t *vals;   // [buckets][2] holder values
    const uint64_t *bits;   // [rows][bpitch] holder bitmaps (at least one row, row 0 of zeros if unused)
    uint32_t shift;         // 64 - log2(buckets)
    uint32_t in_block;      // shift of the second bucket's offset (see buckets_of)
    uint32_t bpitch;        // 64-bit words per bitmap row, a multiple of 12
};

struct Reqs {
    uint32_t n_req;
    const uint32_t *prefill;
    const uint32_t *len;
    const uint64_t *off;
    const uint64_t *hashes;
    uint64_t n_hashes;
};

struct PairOut {
    uint16_t *j;        // [R][D]
    uint8_t *feas;      // [R][D]
    float *score;       // [R][D]
};

// The mixed value of a hash, a multiplicative (Fibonacci) hash of the whole key
// whose top bits serve as an index, and its inverse; 0 stays 0.
__host__ __device__ inline uint64_t mix_hash(uint64_t h) { return h * kGolden; }
__host__ __device__ inline uint64_t unmix_hash(uint64_t x) { return x * kGoldenInv; }

// The two candidate buckets of hash h in a set of 2^b buckets (shift =
// 64 - b): the top b bits of its mixed value, and another bucket, never the
// same one, chosen by the top bits of a second multiplicative hash (the
// multiplier of splitmix64 after an xor-shift).  Both use all 64 bits, so keys
// that agree in part of their bits still get independent pairs.
// In a blocked set (in_block = block_shift(shift)) the second bucket is of the
// same aligned block of 2^11, within 32 KiB, so that a workgroup can build a
// block of the set in LDS.  In a whole set (in_block = shift) it is anywhere:
// the form of resident sets whose mixed values crowd in few blocks, which the
// second bucket then spreads over all of them.  (A chain of two multiplications, with its
// temporaries, in the place of these two cost the kernels that look hashes up
// beside other work more than the lookups: the sequential form's 239 -> 353
// us, a batch of 4,096 16 -> 21 us.)
constexpr uint32_t kBlockLog2 = 11;
__host__ __device__ inline uint32_t block_shift(uint32_t shift) {
    return shift > 64 - kBlockLog2 ? shift : 64 - kBlockLog2;
}
__host__ __device__ inline void buckets_of(uint64_t h, uint32_t shift, uint32_t in_block, uint32_t &b1, uint32_t &b2) {
    b1 = (uint32_t)(mix_hash(h) >> shift);
    b2 = b1 ^ ((uint32_t)(((h ^ (h >> 31)) * kMix64) >> in_block) | 1u);
}

// Row pitch (elements) of the per-(p, d) float2 rows: D rounded up to whole
// 128-byte lines, then to an odd number of lines, so that rows spread over
// all L2 sets instead of aliasing on the sets of a power-of-two stride.
__host__ __device__ inline uint32_t sl_pitch(uint32_t D) {
    uint32_t lines = (D + 15u) / 16u;
    if ((lines & 1u) == 0) ++lines;
    return lines * 16u;
}

// Elements allocated after the last row of the per-(p, d) rows and of the
// leaders' prefix-length table: one group of the widest scoring geometry
// (64 lanes x 6 decodes), so that the scoring kernel's loads for columns
// past the pool stay inside the allocation.
constexpr uint32_t kRowPad = 64u * 6u;

// Holder value of h, by one thread: both candidate buckets' keys, then the
// value of the slot that holds h (most looked-up hashes are held by no
// decode and need no value).
__device__ inline uint32_t holder_lane(const Table &t, uint64_t h) {
    if (h == 0) return kNoHolder;
    uint32_t b1, b2;
    buckets_of(h, t.shift, t.in_block, b1, b2);
    const ulonglong2 k1 = *(const ulonglong2 *)(t.keys + 2 * (uint64_t)b1);
    const ulonglong2 k2 = *(const ulonglong2 *)(t.keys + 2 * (uint64_t)b2);
    const uint64_t slot = k1.x == h ? 2 * (uint64_t)b1 : k1.y == h ? 2 * (uint64_t)b1 + 1
                        : k2.x == h ? 2 * (uint64_t)b2 : k2.y == h ? 2 * (uint64_t)b2 + 1 : ~0ull;
    return slot == ~0ull ? kNoHolder : t.vals[slot];
}

// The same with the second bucket read only where the first is full and does
// not hold h: a hash lies in its second bucket only if its first was full when
// it was placed, and no slot of the set empties again.
__device__ inline uint32_t holder_lane_lean(const Table &t, uint64_t h) {
    if (h == 0) return kNoHolder;
    uint32_t b1, b2;
    buckets_of(h, t.shift, t.in_block, b1, b2);
    uint64_t slot = 2 * (uint64_t)b1;
    ulonglong2 k = *(const ulonglong2 *)(t.keys + slot);
    if (k.x != h && k.y != h && k.x != 0 && k.y != 0) {
        slot = 2 * (uint64_t)b2;
        k = *(const ulonglong2 *)(t.keys + slot);
    }
    return k.x == h ? t.vals[slot] : k.y == h ? t.vals[slot + 1] : kNoHolder;
}

// The shared index: the hashes that two or more decodes hold, with their
// bitmap rows.  One 16-byte slot holds a key and its row, and linear probing
// at a load factor of a sixth to a third finds most keys, and most absences,
// with one load (the whole index takes three, two of them dependent).
struct Shared {
    const u32x4 *b;       // [mask + 1] key (0 = empty), row, 0; null when there is none
    uint32_t shift;       // 64 - log2(slots)
    uint32_t mask;        // slots - 1
};

__device__ inline uint32_t shared_slot(const Shared &t, uint64_t h) { return (uint32_t)((h * kGolden) >> t.shift); }

// The row of h, given the content x of slot i where its probes start.
__device__ inline uint32_t shared_find(const Shared &t, uint64_t h, uint32_t i, u32x4 x) {
    for (;;) {   // ends: there are more slots than keys
        const uint64_t k = ((uint64_t)x.y << 32) | x.x;
        if (k == h) return h == 0 ? kNoHolder : x.z;
        if (k == 0) return kNoHolder;
        i = (i + 1) & t.mask;
        x = t.b[i];
    }
}

// Is h resident on decode d?
__device__ inline bool holds(const Table &t, uint64_t h, uint32_t d) {
    const uint32_t v = holder_lane(t, h);
    if (v == kNoHolder) return false;
    if (v & kHeldOne) return (v & ~kHeldOne) == d;
    return (t.bits[(uint64_t)v * t.bpitch + d / 64u] >> (d % 64u)) & 1ull;
}

// T_queue + T_decode of decode d, scaled by alpha (Sec. IV-B, Eqs. (6)-(7)).
__device__ inline float load_term(const Snap &s, uint32_t d) {
    int64_t q = (int64_t)s.queue[d];
    int64_t beta = (int64_t)s.batch[d];
    int64_t blocked = q - ((int64_t)s.beta_max - beta);
    blocked = blocked < 0 ? 0 : blocked;
    float t_cur = s.t_a + s.t_b * (float)beta;
    float t_next = s.t_a + s.t_b * (float)(beta + 1);
    return s.alpha * ((float)blocked * t_cur + t_next);
}

// The cost of Eq. (5) factored by what each factor depends on.  With
// x = l_r - lambda non-cached tokens (Eq. (2) divided by the bytes per token):
//   s_eff / B_eff(p,d) = x * bpt (1 + n_inflight[tau][p]) / (B_tau (1 - c(p,d)))
// (Eqs. (3)-(4)), so the pair contributes x * spt(p,d) + L_tau, and the decode
// alpha (T_queue + T_decode); feasibility m_d >= bpt x + m_min holds iff
// x < xlim_d = floor((m_d - m_min) / bpt) + 1 (integer, exact).
// Seconds per non-cached token with an explicit in-flight count n.  The
// ablation rungs of the method drop the live congestion (policy 1) or both
// the congestion and the in-flight term (policy 2).
__device__ inline float sec_per_token_n(const Snap &s, uint32_t tau, float n, float c) {
    const float ce = s.policy >= 1 ? 0.0f : c;
    const float ne = s.policy >= 2 ? 0.0f : n;
    return ((float)s.bpt * (1.0f + ne)) / (s.bw[tau] * (1.0f - ce));
}

__device__ inline float sec_per_token(const Snap &s, uint32_t tau, uint32_t p, float c) {
    return sec_per_token_n(s, tau, (float)s.n_inflight[tau * s.P + p], c);
}

// Tier latency by a per-lane tier index, without indexing an array.
__device__ inline float tier_latency(const Snap &s, uint32_t tau) {
    const float lo = (tau & 1u) ? s.lat[1] : s.lat[0];
    const float hi = (tau & 1u) ? s.lat[3] : s.lat[2];
    return (tau & 2u) ? hi : lo;
}

__device__ inline uint64_t feasible_limit(const Snap &s, uint64_t m) {
    if (m < s.m_min) return 0;
    if (s.bpt == 0) return ~0ull;
    return (m - s.m_min) / s.bpt + 1;
}

__device__ inline float pair_score(uint32_t x, float spt, float lat, float base) {
    return fmaf((float)x, spt, lat + base);
}

template <int K>
__device__ inline void topk_insert(uint64_t (&lst)[K], uint64_t x) {
#pragma unroll
    for (int i = 0; i < K; ++i) {
        uint64_t lo = lst[i] < x ? lst[i] : x;
        x = lst[i] < x ? x : lst[i];
        lst[i] = lo;
    }
}

__device__ inline uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) v += __shfl_xor(v, m, kWave);
    return v;
}

// Index of the calling wavefront in its workgroup, as a wave-uniform value
// (so everything derived from it stays in scalar registers).
__device__ inline uint32_t wave_index() {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
}

// Minimum of a 32-bit value over the 64 lanes with DPP row operations
// (quad permutes, row rotates, then the row broadcasts of wave64); every lane
// must be active.  The result is read from lane 63.
__device__ inline uint32_t wave_min_u32_dpp(uint32_t v) {
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x124, 0xF, 0xF, false));  // row_ror 4
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x128, 0xF, 0xF, false));  // row_ror 8
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x142, 0xA, 0xF, false));  // row_bcast 15
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x143, 0xC, 0xF, false));  // row_bcast 31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Minima over the 64 lanes of three values at once (12 VALU instructions
// where three wave_min_u32_dpp take 21).  permlane32_swap exchanges the
// upper half of a with the lower half of b, so one min leaves, in lanes
// 0-31, a's minimum over lanes l and l + 32 and, in lanes 32-63, b's.
// permlane16_swap then exchanges that register's odd rows of 16 lanes with
// c's even rows, and one min gives row 0 a's minimum over lanes i, i + 16,
// i + 32, i + 48, row 2 b's, and rows 1 and 3 c's over the lower and upper
// half.  A DPP minimum within each row finishes all of them: a in lane 0,
// b in lane 32, c the lesser of lanes 16 and 48.  Every lane must be
// active.
template <int CTRL>
__device__ inline uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, CTRL, 0xF, 0xF, false);
}

__device__ inline void wave_min3_u32(uint32_t a, uint32_t b, uint32_t c, uint32_t &ma, uint32_t &mb,
                                     uint32_t &mc) {
    const auto s32 = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    const uint32_t x = min((uint32_t)s32[0], (uint32_t)s32[1]);
    const auto s16 = __builtin_amdgcn_permlane16_swap(x, c, false, false);
    uint32_t z = min((uint32_t)s16[0], (uint32_t)s16[1]);
    z = min(z, dpp_u32<0xB1>(z));    // quad_perm 1,0,3,2
    z = min(z, dpp_u32<0x4E>(z));    // quad_perm 2,3,0,1
    z = min(z, dpp_u32<0x124>(z));   // row_ror 4
    z = min(z, dpp_u32<0x128>(z));   // row_ror 8
    ma = (uint32_t)__builtin_amdgcn_readlane((int)z, 0);
    mb = (uint32_t)__builtin_amdgcn_readlane((int)z, 32);
    mc = min((uint32_t)__builtin_amdgcn_readlane((int)z, 16), (uint32_t)__builtin_amdgcn_readlane((int)z, 48));
}

// Validate request r's header; returns false (and flags) if inconsistent.
__device__ inline bool request_ok(const Reqs &rq, const Snap &s, uint32_t r, uint32_t &p,
                                  uint32_t &len, uint64_t &a, uint32_t &n) {
    p = rq.prefill[r];
    len = rq.len[r];
    a = rq.off[r];
    uint64_t b = rq.off[r + 1];
    if (!(p < s.P && len >= 1 && b >= a && b <= rq.n_hashes)) return false;
    if (b - a != (uint64_t)(len / s.block_tokens)) return false;
    n = (uint32_t)(b - a);
    return true;
}

// Per-call factors of the cost: seconds per token and the constant part
// (tier latency plus load term) for every (p, d), the load term and the
// feasibility limit for every d.  Reads the current snapshot
// (congestion, in-flight counters, queue, batch, free memory).
__global__ __launch_bounds__(256) void derive_kernel(Snap s, float2 *__restrict__ sl, float *__restrict__ dbase,
                                                     uint64_t *__restrict__ dxlim) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t npd = (uint64_t)s.P * s.D;
    if (i < npd) {
        const uint32_t p = (uint32_t)(i / s.D);
        const uint32_t d = (uint32_t)(i - (uint64_t)p * s.D);
        const uint32_t tau = s.tier_map[i] & 3u;
        // the constant part is rounded exactly as latency + load term would
        // be when added after loading both (no contraction into an FMA)
        sl[(uint64_t)p * s.slp + d] =
            make_float2(sec_per_token(s, tau, p, s.util[i]), __fadd_rn(tier_latency(s, tau), load_term(s, d)));
    }
    if (i < s.D) {
        dbase[i] = load_term(s, (uint32_t)i);
        dxlim[i] = feasible_limit(s, s.free_mem[i]);
    }
}

// Two-hop routing (Sec. VIII): the staged route p -> staging store -> d of
// every pair, with hop tiers t1, t2 and congestion u1, u2.  Its transfer
// time is the sum of the hops' (Eqs. (3)-(4) each): seconds per token
// bpt (1 + n_inflight[t1][p]) / (B_t1 (1 - u1)) + bpt / (B_t2 (1 - u2)) (the
// staging store's transfers are not the prefill's in-flight ones) and the
// constant part L_t1 + L_t2 plus the decode's load term.
__global__ __launch_bounds__(256) void derive_route_kernel(Snap s, const uint8_t *__restrict__ t1,
                                                           const float *__restrict__ u1,
                                                           const uint8_t *__restrict__ t2,
                                                           const float *__restrict__ u2, float2 *__restrict__ sr) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t npd = (uint64_t)s.P * s.D;
    if (i >= npd) return;
    const uint32_t p = (uint32_t)(i / s.D);
    const uint32_t d = (uint32_t)(i - (uint64_t)p * s.D);
    const uint32_t a = t1[i] & 3u, b = t2[i] & 3u;
    const float spt = sec_per_token(s, a, p, u1[i]) + sec_per_token_n(s, b, 0.0f, u2[i]);
    sr[(uint64_t)p * s.slp + d] =
        make_float2(spt, __fadd_rn(__fadd_rn(tier_latency(s, a), tier_latency(s, b)), load_term(s, d)));
}

// ---------------------------------------------------------------- batch order
//
// Prefix lengths follow from a batch order that groups equal leading blocks.
// The sort key is 19 bits of the first block hash above 12 bits of the
// complemented run length, so requests that start with the same prefix are
// neighbours in descending length ("hash order").  For neighbours r' -> r
// with a common leading run of L blocks, the first-miss index of r on any
// decode d is j(r', d) whenever that lies inside the common run (blocks
// 0..j(r',d) of r are those of r'), and otherwise it is at least L.  So if
// block L of r is held by no decode (or r has no block L), j(r, d) =
// min(j(r', d), L) exactly, on every decode.
//
// A position whose block L some decode holds is a "leader": its prefix
// lengths are computed from block 0 on every decode (leader kernel).  Every
// other position m then has j(m, d) = min(j(ell, d), L*) with ell the last
// leader before it in hash order and L* the least common run L over the
// positions after ell up to m; with no leader before it, j = 0.  A
// segmented scan over the hash order gives each position its (ell, L*).
// Longest first, a request that is a prefix of its predecessor has L = n_r
// and one that leaves the shared chain first resumes at a block of its own,
// which usually no decode holds, so leaders are about one per shared chain.
//
// Scoring then runs in prefill order (the hash order kept within each
// prefill, a stable radix sort): consecutive requests share their row of
// the snapshot and often their leader, so both are re-read from L1.

constexpr uint32_t kKeyLenBits = 12;             // low key bits: 4095 - min(blocks, 4095)
constexpr uint32_t kKeyEmptyRun = 0x80000000u;   // valid request without blocks
constexpr uint32_t kKeyInvalid = 0xFFFFFFFFu;
constexpr uint32_t kNoLead = 0xFFFFFFFFu;        // no leader before the position
constexpr uint32_t kLeadOver = 0xFFFFFFFEu;      // a leader beyond the leader table's capacity
constexpr uint32_t kNoCap = 0xFFFFFFFFu;         // L* of a leader itself (no cap)

// Segmented-scan element of a hash-order position: leader slot (or kNoLead
// for a non-leader) in the high word, common run L (kNoCap for a leader) in
// the low word.  Combining keeps the later leader, else the earlier leader
// with the smaller L; the combination is associative.
__host__ __device__ inline uint64_t seg_elem(uint32_t slot, uint32_t l) { return ((uint64_t)slot << 32) | l; }
struct SegOp {
    __host__ __device__ uint64_t operator()(uint64_t a, uint64_t b) const {
        if ((uint32_t)(b >> 32) != kNoLead) return b;
        const uint32_t la = (uint32_t)a, lb = (uint32_t)b;
        return (a & 0xFFFFFFFF00000000ull) | (la < lb ? la : lb);
    }
};

// The identity of SegOp: no leader, no cap.
constexpr uint64_t kSegIdentity = ((uint64_t)kNoLead << 32) | kNoCap;
__device__ inline uint64_t seg_op(uint64_t a, uint64_t b) { return SegOp()(a, b); }

// A leader: where its blocks' holder values start in hv (from block 0, up
// to the first block no decode holds; m = kNoPre if they did not fit), and
// its hash run for lookups otherwise.
struct alignas(16) Lead {
    uint64_t a;      // offset of the hash run
    uint64_t hoff;   // offset of the holder values
    uint32_t n;      // hashed blocks
    uint32_t m;      // stored holder values, or kNoPre
    uint32_t pad[2];
};
constexpr uint32_t kNoPre = 0xFFFFFFFFu;

// Token counts below 2^24 are integers that fp32 holds exactly: requests
// shorter than that are scored in fp32 with results identical to integer
// arithmetic, longer ones in integers.
constexpr uint32_t kExactTok = 1u << 24;

// A request by hash-order position: its prefill row and length.
struct Pre {
    uint32_t row;    // byte offset of the request's row of derived (p, d) values, p * slp * 8
    uint32_t len;    // input tokens
};

// One request in scoring order: the part every scoring step reads (one
// 16-byte scalar load) ...
struct alignas(16) Hot {
    uint32_t row;    // byte offset of the prefill row, as in Pre
    uint32_t lrow;   // byte offset of the leader's row of B_tok * j in the leader
                     // table; the all-zero row when there is no leader
    uint32_t len;    // input tokens, fp32 bits
    uint32_t lams;   // B_tok * L* (+inf for a leader itself), fp32 bits; negative:
                     // match this request on its own, in integers
};
constexpr uint32_t kHotPad = 2;   // records past the last position, read ahead by the scan

// ... and its index in the caller's batch (where its result goes, and its
// hash run and length when it is matched on its own).
struct Cold {
    uint32_t r;
};

struct Order {
    const Hot *hot;           // [n_valid + kHotPad] scoring-order request records
    const Cold *cold;         // [n_req]
    const float *lam;         // [leader rows][D] B_tok * prefix length of each leader on each decode
    const uint32_t *hv;       // holder values of the leaders' blocks
    const uint32_t *n_valid;  // valid requests (they sort first)
    uint32_t lead_cap;        // leaders the table takes in this call
};

// Validate each request and build its sort key, one thread per request.
// A request of more than max_blocks blocks is invalid (every call passes
// 2^32 - 1: runs of any length are scored).  A block hash 0 needs no
// check: no resident set holds it (cache loads reject it), so it is a miss
// on every decode, as the prefix definition gives.  vals (the input
// positions, for rocPRIM's sort) may be null.  Thread 0 clears the
// holder-value and leader counters of the order kernel.  An invalid
// request's outputs (index -1, score NaN) are written here when out_idx is
// given.
__global__ __launch_bounds__(256) void prep_kernel(Snap s, Reqs rq, uint32_t max_blocks, uint32_t *__restrict__ keys,
                                                   uint32_t *__restrict__ vals, uint32_t *__restrict__ err,
                                                   unsigned long long *__restrict__ hv_used,
                                                   unsigned int *__restrict__ n_lead, uint32_t k_out,
                                                   int32_t *__restrict__ out_idx, float *__restrict__ out_score) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r == 0) {
        *hv_used = 0;
        *n_lead = 0;
    }
    bool bad = false;
    if (r < rq.n_req) {
        uint32_t p, len, n;
        uint64_t a;
        const bool ok = request_ok(rq, s, r, p, len, a, n) && n <= max_blocks;
        uint32_t key = kKeyInvalid;
        if (ok) {
            if (n == 0) {
                key = kKeyEmptyRun;
            } else {
                const uint32_t top = (uint32_t)((rq.hashes[a] * kGolden) >> 32);
                key = ((top >> 13) << kKeyLenBits) | (4095u - (n < 4095u ? n : 4095u));
            }
        }
        keys[r] = key;
        if (vals) vals[r] = r;
        bad = !ok;
        if (bad && out_idx) {
            // an invalid request is answered here (the scoring kernel skips it)
            for (uint32_t q = 0; q < k_out; ++q) {
                out_idx[(uint64_t)r * k_out + q] = -1;
                out_score[(uint64_t)r * k_out + q] = __builtin_nanf("");
            }
        }
    }
    if (__ballot(bad) && (threadIdx.x % kWave) == 0) atomicOr(err, kErrRequest);
}

// Per hash-order position i (G lanes, G divides 64): the common leading run
// L with the previous position (G blocks compared per step, their loads
// issued together), whether the position is a leader (some decode holds its
// block L), and for a leader a slot of the leader table and room for the
// holder values of its blocks (in hv, from a shared counter; filled by
// lead_holder_kernel).  Writes the prefill sort key and the scoring record
// of i, and the number of valid requests (valid keys sort first): the last
// valid position writes it, or position 0 writes 0.  Invalid positions sort
// after every prefill (key P).
//
// The segmented scan of the positions' elements (leader slot, L) is fused
// here, in two levels: each workgroup (kOrderPos positions, one tile) scans
// its own elements and writes, for each position, the inclusive combination
// within the tile (seg) and the tile's total (agg[tile]).
// tile_prefix_kernel turns the totals into exclusive tile prefixes, and the
// record writers combine a position's tile prefix with its in-tile value.
// (A single-pass look-back over tiles was slower here: a tile's prefix can
// be published only a device-scope load round-trip after its predecessor's,
// far slower than tiles complete.)
constexpr uint32_t kLcpLanes = 4;                  // lanes per hash-order position
constexpr uint32_t kOrderPos = 256 / kLcpLanes;    // hash-order positions per order workgroup

// 64-bit lane shuffle up by `off` lanes (within the wavefront).
__device__ inline uint64_t shfl_up_u64(uint64_t v, uint32_t off) {
    const uint32_t lo = (uint32_t)__shfl_up((int)(uint32_t)v, off, kWave);
    const uint32_t hi = (uint32_t)__shfl_up((int)(uint32_t)(v >> 32), off, kWave);
    return ((uint64_t)hi << 32) | lo;
}

template <uint32_t G>
__global__ __launch_bounds__(256) void order_kernel(Reqs rq, uint32_t P, uint32_t slp, uint32_t bt,
                                                    const uint32_t *__restrict__ perm,
                                                    const uint32_t *__restrict__ sorted_keys, Table t,
                                                    uint32_t reuse, uint64_t *__restrict__ seg,
                                                    uint64_t *__restrict__ agg,
                                                    uint32_t *__restrict__ pkey, uint32_t *__restrict__ pval,
                                                    Pre *__restrict__ hrec, Cold *__restrict__ crec,
                                                    Lead *__restrict__ lead, uint32_t lead_cap,
                                                    unsigned int *__restrict__ n_lead, uint64_t hv_cap,
                                                    unsigned long long *__restrict__ hv_used,
                                                    uint32_t *__restrict__ n_valid) {
    static_assert(G * kOrderPos == 256, "positions per workgroup");
    __shared__ uint64_t wtot[kWavesPerBlock];
    const uint32_t sub = threadIdx.x % G;
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t seg0 = lane - sub;   // first lane of this position's lanes
    const uint64_t i = (uint64_t)blockIdx.x * kOrderPos + threadIdx.x / G;
    const bool inb = i < (uint64_t)rq.n_req;
    const bool valid = inb && sorted_keys[i] < kKeyInvalid;
    const uint32_t r = inb ? perm[i] : 0u;
    uint64_t e = kSegIdentity;   // this position's scan element (lane sub == 0)
    if (inb && sub == 0) {
        if (valid && (i + 1 == rq.n_req || sorted_keys[i + 1] >= kKeyInvalid)) *n_valid = (uint32_t)(i + 1);
        if (i == 0 && !valid) *n_valid = 0;
        if (pval) pval[i] = (uint32_t)i;
        if (!valid) {
            e = seg_elem(kNoLead, 0);
            pkey[i] = P;
            hrec[i] = Pre{0, 0};
            crec[i] = Cold{r};
        }
    }
    // this position's run, and the previous position's: from the lanes G
    // below (one wavefront holds kWave / G consecutive positions), or, for
    // the wavefront's first position, loaded
    uint64_t a = 0, nr = 0;
    if (valid) {
        a = rq.off[r];
        nr = rq.off[r + 1] - a;
    }
    const uint32_t pg = lane / G;
    const uint32_t key = valid ? sorted_keys[i] : kKeyInvalid;
    uint32_t kq = (uint32_t)__shfl_up((int)key, G, kWave);
    uint64_t b = shfl_up_u64(a, G), nq = shfl_up_u64(nr, G);
    if (pg == 0 && valid && i > 0) {
        kq = sorted_keys[i - 1];
        const uint32_t q = perm[i - 1];
        b = rq.off[q];
        nq = rq.off[q + 1] - b;
    }
    // keys that differ in their first-block hash bits have different first
    // blocks: nothing in common
    const bool cmp = valid && i > 0 && reuse && (key >> kKeyLenBits) == (kq >> kKeyLenBits);
    const uint64_t m = cmp ? (nr < nq ? nr : nq) : 0;
    uint64_t l = m;
    {
        // Lock-step over the wavefront: each lane loads U consecutive blocks
        // of its own run per step (their loads issued together) while its
        // position or the next one is still comparing, and takes the
        // previous position's blocks from the lanes G below; the first
        // differing block is the lowest lane's first stop.
        constexpr uint32_t U = 2;
        bool act = m > 0;
        for (uint64_t base = 0;; base += (uint64_t)G * U) {
            if (!__any(act)) break;
            const bool act_next = (bool)__shfl_down((int)act, G, kWave) && pg + 1 < (uint32_t)kWave / G;
            const bool need = act || act_next;
            const uint64_t x0 = base + (uint64_t)sub * U;
            uint64_t hr[U], hq[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) hr[u] = (need && x0 + u < nr) ? rq.hashes[a + x0 + u] : 0ull;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) hq[u] = shfl_up_u64(hr[u], G);
            if (pg == 0) {
#pragma unroll
                for (uint32_t u = 0; u < U; ++u) hq[u] = (act && x0 + u < m) ? rq.hashes[b + x0 + u] : 1ull;
            }
            uint32_t ls = U;   // this lane's first stop (U: none); blocks at m and beyond stop
#pragma unroll
            for (int u = (int)U - 1; u >= 0; --u)
                if (x0 + u >= m || hr[u] != hq[u]) ls = (uint32_t)u;
            const uint32_t bits =
                (uint32_t)(__ballot(act && ls < U) >> seg0) & (uint32_t)((1ull << G) - 1);
            if (act && bits) {
                const uint32_t fl = (uint32_t)__builtin_ctz(bits);
                const uint32_t lsf = (uint32_t)__shfl((int)ls, (int)(seg0 + fl), kWave);
                const uint64_t first = base + (uint64_t)fl * U + lsf;
                l = first < m ? first : m;
                act = false;
            }
            if (base + (uint64_t)G * U >= m) act = false;
        }
    }
    if (valid) {
        if (sub == 0) {
            // a leader if some decode holds block L
            const uint32_t vl = l < nr ? holder_lane(t, rq.hashes[a + l]) : kNoHolder;
            e = seg_elem(kNoLead, (uint32_t)l);
            if (vl != kNoHolder) {
                const unsigned int slot = atomicAdd(n_lead, 1u);
                if (slot >= lead_cap) {
                    e = seg_elem(kLeadOver, kNoCap);
                } else {
                    e = seg_elem(slot, kNoCap);
                    const unsigned long long o = atomicAdd(hv_used, (unsigned long long)nr);
                    Lead ld;
                    ld.a = a;
                    ld.hoff = o;
                    ld.n = (uint32_t)nr;
                    ld.m = o + nr <= hv_cap ? 0u : kNoPre;   // filled by lead_holder_kernel
                    ld.pad[0] = ld.pad[1] = 0;
                    lead[slot] = ld;
                }
            }
            pkey[i] = rq.prefill[r];
            hrec[i] = Pre{rq.prefill[r] * slp * (uint32_t)sizeof(float2),   // < 2^32 (checked at load)
                          rq.len[r]};
            crec[i] = Cold{r};
        }
    }
    // the tile's scan: the wavefront's positions (lanes sub == 0, G apart)
    // by shuffles, then the wavefronts' totals in order
#pragma unroll
    for (uint32_t off = G; off < (uint32_t)kWave; off <<= 1) {
        const uint64_t prev = shfl_up_u64(e, off);
        if (lane >= off) e = seg_op(prev, e);
    }
    const uint32_t w = threadIdx.x / kWave;
    if (lane == kWave - G) wtot[w] = e;
    __syncthreads();
    uint64_t pre = kSegIdentity;
    for (uint32_t q = 0; q < w; ++q) pre = seg_op(pre, wtot[q]);
    e = seg_op(pre, e);
    if (inb && sub == 0) seg[i] = e;
    if (threadIdx.x == 0) {
        uint64_t tot = kSegIdentity;
#pragma unroll
        for (uint32_t q = 0; q < kWavesPerBlock; ++q) tot = seg_op(tot, wtot[q]);
        agg[blockIdx.x] = tot;
    }
}

// Exclusive prefixes of the order workgroups' tile totals, in place: one
// workgroup of kPrefixThreads, kPrefixThreads * kPrefixPer totals per round
// (one round up to 2^24 requests), each thread combining its consecutive
// totals, the threads' results scanned by shuffles and then across the
// wavefronts, with the running prefix of earlier rounds.
constexpr uint32_t kPrefixThreads = 1024;
constexpr uint32_t kPrefixWaves = kPrefixThreads / kWave;
constexpr uint32_t kPrefixPer = 16;
static_assert(kPrefixPer % 2 == 0, "totals move in pairs");
__global__ __launch_bounds__(kPrefixThreads) void tile_prefix_kernel(uint64_t *__restrict__ agg, uint32_t n) {
    __shared__ uint64_t wtot[kPrefixWaves];
    __shared__ uint64_t carry_s;
    const uint32_t tid = threadIdx.x, lane = tid % kWave, w = tid / kWave;
    uint64_t carry = kSegIdentity;
    for (uint64_t r0 = 0; r0 < n; r0 += (uint64_t)kPrefixThreads * kPrefixPer) {
        const uint64_t b0 = r0 + (uint64_t)tid * kPrefixPer;
        // a thread's totals are consecutive: whole runs move in 16-byte
        // pieces (half the requests of 8-byte ones), the tail one by one
        const bool whole = b0 + kPrefixPer <= n;
        uint64_t v[kPrefixPer];
        if (whole) {
            const u64x2 *src = (const u64x2 *)(agg + b0);   // 16-byte aligned: b0 is a multiple of 16
#pragma unroll
            for (uint32_t u = 0; u < kPrefixPer / 2; ++u) {
                const u64x2 x = src[u];
                v[2 * u] = x.x;
                v[2 * u + 1] = x.y;
            }
        } else {
#pragma unroll
            for (uint32_t u = 0; u < kPrefixPer; ++u) v[u] = b0 + u < n ? agg[b0 + u] : kSegIdentity;
        }
        uint64_t tot = kSegIdentity;
#pragma unroll
        for (uint32_t u = 0; u < kPrefixPer; ++u) tot = seg_op(tot, v[u]);
        // inclusive scan of the threads' totals within the wavefront
        uint64_t inc = tot;
#pragma unroll
        for (uint32_t off = 1; off < (uint32_t)kWave; off <<= 1) {
            const uint64_t prev = shfl_up_u64(inc, off);
            if (lane >= off) inc = seg_op(prev, inc);
        }
        const uint64_t prev1 = shfl_up_u64(inc, 1);
        if (lane == kWave - 1) wtot[w] = inc;
        __syncthreads();
        uint64_t pre = carry;
        for (uint32_t q = 0; q < w; ++q) pre = seg_op(pre, wtot[q]);
        // this thread's first total's exclusive prefix
        uint64_t run = lane > 0 ? seg_op(pre, prev1) : pre;
        uint64_t ex[kPrefixPer];   // the exclusive prefixes
#pragma unroll
        for (uint32_t u = 0; u < kPrefixPer; ++u) {
            ex[u] = run;
            run = seg_op(run, v[u]);
        }
        if (whole) {
            u64x2 *dst = (u64x2 *)(agg + b0);
#pragma unroll
            for (uint32_t u = 0; u < kPrefixPer / 2; ++u) {
                u64x2 x;
                x.x = ex[2 * u];
                x.y = ex[2 * u + 1];
                dst[u] = x;
            }
        } else {
#pragma unroll
            for (uint32_t u = 0; u < kPrefixPer; ++u)
                if (b0 + u < n) agg[b0 + u] = ex[u];
        }
        if (tid == kPrefixThreads - 1) carry_s = run;
        __syncthreads();
        carry = carry_s;
        __syncthreads();
    }
}

// The scanned element (last leader slot, L*) of hash-order position i: its
// tile's exclusive prefix combined with its inclusive value in the tile.
__device__ inline uint64_t scanned_at(const uint64_t *seg, const uint64_t *tpre, uint64_t i) {
    return seg_op(tpre[i / kOrderPos], seg[i]);
}

// Holder values of every leader's blocks from block 0 up to the first
// block no decode holds: one wavefront per leader (looping over leaders,
// whose count is read from device memory), lanes over blocks.
__global__ __launch_bounds__(kBlock) void lead_holder_kernel(Table t, const uint64_t *__restrict__ hashes,
                                                             Lead *__restrict__ lead,
                                                             const unsigned int *__restrict__ n_lead,
                                                             uint32_t lead_cap, uint32_t *__restrict__ hv) {
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t nl_all = *n_lead;
    const uint32_t nl = nl_all < lead_cap ? nl_all : lead_cap;
    const uint32_t nw = gridDim.x * kWavesPerBlock;
    for (uint32_t slot = blockIdx.x * kWavesPerBlock + wave_index(); slot < nl; slot += nw) {
        const Lead ld = lead[slot];
        if (ld.m == kNoPre) continue;   // no room: the leader kernel looks its blocks up
        uint32_t m = ld.n;
        for (uint32_t k0 = 0; k0 < ld.n; k0 += kWave) {
            const uint32_t k = k0 + lane;
            uint32_t hk = kNoHolder;
            if (k < ld.n) {
                hk = holder_lane(t, hashes[ld.a + k]);
                hv[ld.hoff + k] = hk;
            }
            const uint64_t none = __ballot(k < ld.n && hk == kNoHolder);
            if (none) {
                m = k0 + (uint32_t)__builtin_ctzll(none);
                break;
            }
        }
        if (lane == 0) lead[slot].m = m;
    }
}

// The scoring record of a request from its prefill row and length and its
// scan element (leader slot, L*).
__device__ inline Hot make_hot(Pre pr, uint64_t e, uint32_t bt, uint32_t lstride, uint32_t zrow) {
    const uint32_t ls = (uint32_t)e, slot = (uint32_t)(e >> 32);
    const bool own = slot == kLeadOver || pr.len >= kExactTok;
    Hot o;
    o.row = pr.row;
    o.lrow = (slot < kLeadOver && !own) ? slot * lstride : zrow;
    o.len = __float_as_uint((float)pr.len);
    // ls <= n_r, so bt * ls <= len
    o.lams = own ? __float_as_uint(-1.0f)
                 : ls == kNoCap ? __float_as_uint(__builtin_inff()) : __float_as_uint((float)(bt * ls));
    return o;
}

// Scoring-order records: position k of the prefill order holds hash-order
// position pord[k], whose record takes its leader row and B_tok * L* from
// the scan (lstride: bytes per leader row; zrow: byte offset of the
// all-zero row).  A request whose leader did not fit the leader table, or
// of 2^24 tokens or more, is marked to be matched on its own.  Positions
// past the batch (kHotPad of them) get a record that the scoring kernel
// may read ahead but never scores (row 0, no leader).  With hotr, each
// request's record is also written at its index in the batch (the ranking
// sweep reads records in batch order).
__global__ __launch_bounds__(256) void assemble_kernel(uint32_t n_req, uint32_t bt, uint32_t lstride, uint32_t zrow,
                                                       const uint32_t *__restrict__ pord,
                                                       const uint64_t *__restrict__ seg,
                                                       const uint64_t *__restrict__ tpre,
                                                       const Pre *__restrict__ hrec, const Cold *__restrict__ crec,
                                                       Hot *__restrict__ hot, Cold *__restrict__ cold,
                                                       Hot *__restrict__ hotr) {
    const uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (uint64_t)n_req + kHotPad) return;
    if (k >= n_req) {
        hot[k] = Hot{0, zrow, 0, 0};
        return;
    }
    const uint32_t i = pord[k];
    const Hot rec = make_hot(hrec[i], scanned_at(seg, tpre, i), bt, lstride, zrow);
    const Cold c = crec[i];
    hot[k] = rec;
    cold[k] = c;
    if (hotr) hotr[c.r] = rec;
}

// The scoring records by batch index alone (the sequential form orders its
// chains itself and scores nothing in prefill order).
__global__ __launch_bounds__(256) void records_kernel(uint32_t n_req, uint32_t bt, uint32_t lstride, uint32_t zrow,
                                                      const uint64_t *__restrict__ seg,
                                                      const uint64_t *__restrict__ tpre,
                                                      const Pre *__restrict__ hrec, const Cold *__restrict__ crec,
                                                      Hot *__restrict__ hotr) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_req) hotr[crec[i].r] = make_hot(hrec[i], scanned_at(seg, tpre, i), bt, lstride, zrow);
}

// ---------------------------------------------------------------- batch sorts
//
// Stable LSD radix sort for the batch orders (batches of kSortMinN + 1 to
// kSortMaxN): tiles of TILE positions (sort_tile: 1,024 up to
// kSortSmallTileN positions, so that a batch of a few hundred thousand
// still spreads over every CU, else 4,096, whose digits leave in longer
// runs), one workgroup each, in passes of at most kSortMaxBits digit bits.
// A pass takes three kernels:
// sort_count_kernel counts each tile's digits into cnt[tile][digit];
// sort_colscan_kernel turns every digit's column into exclusive offsets
// over the tiles (in place) and writes the digit totals;
// sort_scatter_kernel ranks the tile's elements (each wavefront a quarter
// of the tile, 64 at a time, equal digits ranked by lane masks), stages
// them in LDS in output order and writes them out in that order, so that
// the elements of one digit leave as a contiguous run.  Equal keys keep
// their order (stable), which the prefill order relies on.
constexpr uint32_t kSortTile = 4096;           // the large tile
constexpr uint32_t kSortSmallTile = 1024;      // the small tile
constexpr uint64_t kSortSmallTileN = 1ull << 19;   // largest batch sorted in small tiles (512 of them)
constexpr uint32_t kSortMaxBits = 11;   // widest pass: the prefill order of up to 2,047 prefills in one
constexpr uint32_t kSortMaxBins = 1u << kSortMaxBits;
constexpr uint32_t kSortPassBits = 8;   // passes of the hash order and the general pair sort (faster per bit)
constexpr uint32_t kSortBinsPer = kSortMaxBins / kBlock;   // digits per thread at the widest pass
constexpr uint32_t kPrefillMaxBits = 16;   // prefill keys of more bits: rocPRIM's sort and a gather
constexpr uint64_t kSortMaxN = 1ull << 24;
constexpr uint64_t kSortMinN = 1ull << 16;   // smaller batches: rocPRIM (fewer launches)
constexpr uint64_t kForkMinN = 1ull << 16;   // batches from which a selection forks its second stream
static_assert(kSortBinsPer * kBlock == kSortMaxBins, "digits split evenly over the threads");

// Tile size of the batch sorts for n positions.
inline uint32_t sort_tile(uint64_t n) { return n <= kSortSmallTileN ? kSortSmallTile : kSortTile; }

template <uint32_t TILE>
__global__ __launch_bounds__(kBlock) void sort_count_kernel(const uint32_t *__restrict__ keys, uint32_t n,
                                                            uint32_t shift, uint32_t bits,
                                                            uint32_t *__restrict__ cnt) {
    constexpr uint32_t kPer = TILE / kBlock;   // positions per thread
    __shared__ uint32_t h[kSortMaxBins];
    const uint32_t bins = 1u << bits, mask = bins - 1;
    const uint32_t tid = threadIdx.x;
    for (uint32_t b = tid; b < bins; b += kBlock) h[b] = 0;
    __syncthreads();
    const uint64_t e0 = (uint64_t)blockIdx.x * TILE + tid;
    uint32_t kr[kPer];   // the thread's keys, all loads issued first
#pragma unroll
    for (uint32_t x = 0; x < kPer; ++x) {
        const uint64_t e = e0 + (uint64_t)x * kBlock;
        kr[x] = e < n ? keys[e] : 0u;
    }
#pragma unroll
    for (uint32_t x = 0; x < kPer; ++x)
        if (e0 + (uint64_t)x * kBlock < n) atomicAdd(h + ((kr[x] >> shift) & mask), 1u);
    __syncthreads();
    for (uint32_t b = tid; b < bins; b += kBlock) cnt[(uint64_t)blockIdx.x * bins + b] = h[b];
}

// Inclusive prefix sum over the 64 lanes of a wavefront.
__device__ inline uint32_t wave_incl_scan(uint32_t v) {
    const uint32_t lane = threadIdx.x % kWave;
#pragma unroll
    for (uint32_t off = 1; off < (uint32_t)kWave; off <<= 1) {
        const uint32_t u = __shfl_up(v, off, kWave);
        if (lane >= off) v += u;
    }
    return v;
}

// One workgroup per digit: the exclusive offsets of the digit's column
// over the tiles (in place) and the digit total.  Thread t takes kColPer
// consecutive tiles (fewer at the end), sums them, and the workgroup scans
// the sums.
constexpr uint32_t kColPer = (uint32_t)(kSortMaxN / kSortTile / kBlock);
static_assert(kColPer * kBlock * kSortTile == kSortMaxN, "column scan covers the largest batch");
static_assert(kSortSmallTileN / kSortSmallTile <= (uint64_t)kColPer * kBlock, "and the most small tiles");
__global__ __launch_bounds__(kBlock) void sort_colscan_kernel(uint32_t *__restrict__ cnt, uint32_t ntile,
                                                              uint32_t bits, uint32_t *__restrict__ tot) {
    __shared__ uint32_t wsum[kWavesPerBlock];
    const uint32_t bins = 1u << bits, b = blockIdx.x, t = threadIdx.x;
    const uint32_t per = (ntile + kBlock - 1) / kBlock;   // <= kColPer
    const uint32_t t0 = t * per;
    uint32_t c[kColPer];
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t u = 0; u < kColPer; ++u) {
        c[u] = (u < per && t0 + u < ntile) ? cnt[(uint64_t)(t0 + u) * bins + b] : 0u;
        sum += c[u];
    }
    const uint32_t incl = wave_incl_scan(sum);
    if (t % kWave == kWave - 1) wsum[t / kWave] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (uint32_t q = 0; q < t / kWave; ++q) run += wsum[q];
#pragma unroll
    for (uint32_t u = 0; u < kColPer; ++u) {
        if (u < per && t0 + u < ntile) cnt[(uint64_t)(t0 + u) * bins + b] = run;
        run += c[u];
    }
    if (t == kBlock - 1) tot[b] = run;
}

// Exclusive prefix sum of v[0, bins) in LDS, in place, by the whole
// workgroup: thread t takes consecutive digits t*per .. t*per + per - 1
// (per = bins / kBlock, at least 1), the wavefronts scan the threads' sums
// with lane shuffles, then the four wavefront totals are added.
__device__ inline void lds_exclusive_scan(uint32_t *v, uint32_t bins) {
    __shared__ uint32_t wsum[kWavesPerBlock];
    const uint32_t t = threadIdx.x;
    const uint32_t per = bins > (uint32_t)kBlock ? bins / kBlock : 1u;
    const uint32_t b0 = t * per;
    uint32_t loc[kSortBinsPer];
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t u = 0; u < kSortBinsPer; ++u) {
        loc[u] = (u < per && b0 + u < bins) ? v[b0 + u] : 0u;
        sum += loc[u];
    }
    const uint32_t incl = wave_incl_scan(sum);
    if (t % kWave == kWave - 1) wsum[t / kWave] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (uint32_t q = 0; q < t / kWave; ++q) run += wsum[q];
#pragma unroll
    for (uint32_t u = 0; u < kSortBinsPer; ++u) {
        if (u < per && b0 + u < bins) v[b0 + u] = run;
        run += loc[u];
    }
    __syncthreads();
}

// Lanes of the calling wavefront in `valid` whose digit equals this lane's
// (the digit's bits compared one ballot at a time).
__device__ inline uint64_t digit_peers(uint32_t d, uint32_t bits, uint64_t valid) {
    uint64_t m = valid;
    for (uint32_t j = 0; j < bits; ++j) {
        const bool bit = (d >> j) & 1u;
        const uint64_t b = __builtin_amdgcn_ballot_w64(bit);
        m &= bit ? b : ~b;
    }
    return m;
}

// Scatter of one pass.  The values are vin's, or the input positions when
// vin is null.  ASSEMBLE: the values are hash-order positions and each
// element writes its scoring records (from hrec, the scan and crec at that
// position) at its output position (and, with hotr, at the request's index
// in the batch); the kHotPad records past the batch are written too.
// Otherwise (key, value) pairs go to kout / vout.
template <bool ASSEMBLE, uint32_t TILE>
__global__ __launch_bounds__(kBlock) void sort_scatter_kernel(const uint32_t *__restrict__ kin,
                                                              const uint32_t *__restrict__ vin, uint32_t n,
                                                              uint32_t shift, uint32_t bits,
                                                              const uint32_t *__restrict__ cnt,
                                                              const uint32_t *__restrict__ tot,
                                                              uint32_t *__restrict__ kout, uint32_t *__restrict__ vout,
                                                              const Pre *__restrict__ hrec,
                                                              const uint64_t *__restrict__ seg,
                                                              const uint64_t *__restrict__ tpre,
                                                              const Cold *__restrict__ crec, uint32_t bt,
                                                              uint32_t lstride, uint32_t zrow, Hot *__restrict__ hot,
                                                              Cold *__restrict__ cold, Hot *__restrict__ hotr) {
    constexpr uint32_t kPer = TILE / kBlock;                  // positions per thread
    constexpr uint32_t kQuarter = TILE / kWavesPerBlock;      // positions per wavefront
    constexpr uint32_t kSteps = kQuarter / kWave;             // 64-position steps of a wavefront
    __shared__ uint32_t bb[kSortMaxBins];                     // the tile's first output position per digit
    __shared__ uint32_t hist[kWavesPerBlock][kSortMaxBins];   // per-wavefront counts, then their prefixes
    __shared__ uint32_t toff[kSortMaxBins];                   // first staging slot per digit
    __shared__ uint32_t sk[TILE], sv[TILE];                   // keys and values in output order
    const uint32_t bins = 1u << bits, mask = bins - 1;
    const uint32_t tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
    const uint64_t t0 = (uint64_t)blockIdx.x * TILE;
    for (uint32_t b = tid; b < bins; b += kBlock) bb[b] = tot[b];
    for (uint32_t b = lane; b < bins; b += kWave) hist[w][b] = 0;
    __syncthreads();
    lds_exclusive_scan(bb, bins);   // the digits' first output positions
    for (uint32_t b = tid; b < bins; b += kBlock) bb[b] += cnt[(uint64_t)blockIdx.x * bins + b];
    if (ASSEMBLE && blockIdx.x == 0 && tid < kHotPad) hot[(uint64_t)n + tid] = Hot{0, zrow, 0, 0};
    // this wavefront's quarter of the tile: keys and values, loads first
    const uint64_t e0 = t0 + (uint64_t)w * kQuarter + lane;
    uint32_t kr[kSteps], vr[kSteps], rk[kSteps];
#pragma unroll
    for (uint32_t x = 0; x < kSteps; ++x) {
        const uint64_t e = e0 + (uint64_t)x * kWave;
        kr[x] = e < n ? kin[e] : 0u;
        vr[x] = e < n ? (vin ? vin[e] : (uint32_t)e) : 0u;
    }
    __syncthreads();
    // rank within the wavefront's quarter, step by step
#pragma unroll
    for (uint32_t x = 0; x < kSteps; ++x) {
        const bool valid = e0 + (uint64_t)x * kWave < n;
        const uint32_t d = (kr[x] >> shift) & mask;
        const uint64_t peers = digit_peers(d, bits, __builtin_amdgcn_ballot_w64(valid));
        const uint32_t at = hist[w][d];
        if (valid && lane == (uint32_t)__builtin_ctzll(peers)) hist[w][d] = at + (uint32_t)__builtin_popcountll(peers);
        rk[x] = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
    }
    __syncthreads();
    // per digit: the wavefronts' prefixes (in place) and the tile count
    for (uint32_t b = tid; b < bins; b += kBlock) {
        uint32_t run = 0;
#pragma unroll
        for (uint32_t q = 0; q < kWavesPerBlock; ++q) {
            const uint32_t c = hist[q][b];
            hist[q][b] = run;
            run += c;
        }
        toff[b] = run;
    }
    __syncthreads();
    lds_exclusive_scan(toff, bins);   // the digits' first staging slots
    // stage in output order
#pragma unroll
    for (uint32_t x = 0; x < kSteps; ++x) {
        if (e0 + (uint64_t)x * kWave < n) {
            const uint32_t d = (kr[x] >> shift) & mask;
            const uint32_t pos = toff[d] + hist[w][d] + rk[x];
            sk[pos] = kr[x];
            sv[pos] = vr[x];
        }
    }
    __syncthreads();
    // write out in output order: one digit's elements are consecutive
    const uint32_t nt = n - t0 < (uint64_t)TILE ? (uint32_t)(n - t0) : TILE;
#pragma unroll
    for (uint32_t x = 0; x < kPer; ++x) {
        const uint32_t j = x * kBlock + tid;
        if (j < nt) {
            const uint32_t k = sk[j];
            const uint32_t d = (k >> shift) & mask;
            const uint32_t o = bb[d] + (j - toff[d]);
            if (ASSEMBLE) {
                const uint32_t e = sv[j];
                const Hot rec = make_hot(hrec[e], scanned_at(seg, tpre, e), bt, lstride, zrow);
                const Cold c = crec[e];
                hot[o] = rec;
                cold[o] = c;
                if (hotr) hotr[c.r] = rec;
            } else {
                kout[o] = k;
                vout[o] = sv[j];
            }
        }
    }
}

// Read-only data that is uniform across a wavefront (request records, hash
// runs) is read through the constant address space, which the compiler
// serves with scalar loads into SGPRs.
template <typename T>
using cptr = const __attribute__((address_space(4))) T *;

template <typename T>
__device__ inline cptr<T> as_const(const T *p) {
    return (cptr<T>)(const __attribute__((address_space(4))) void *)(uintptr_t)p;
}

__device__ inline Hot load_hot(const Hot *base, uint32_t i) {
    const cptr<uint32_t> w = as_const((const uint32_t *)(base + i));
    Hot x;
    x.row = w[0];
    x.lrow = w[1];
    x.len = w[2];
    x.lams = w[3];
    return x;
}

__device__ inline Cold load_cold(const Cold *base, uint32_t i) {
    return Cold{as_const((const uint32_t *)base)[i]};
}

// Lane masks of a wavefront: ballot turns a per-lane predicate into a
// uniform 64-bit mask (held in scalar registers), in_mask reads a lane's
// bit back as a predicate.  Per-column "alive" and "need" sets are kept as
// masks so that their tests and combinations are scalar operations.
using lmask = uint64_t;

__device__ inline lmask ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ inline bool in_mask(lmask m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// v_writelane: lane `l` (uniform) of `old` takes the uniform value `v`, the
// other lanes keep theirs.  The compiler offers no builtin for it, so the
// intrinsic is declared by its name.
extern "C" __device__ int amdgcn_writelane(int v, int l, int old) __asm("llvm.amdgcn.writelane.i32");
__device__ inline uint32_t write_lane(uint32_t v, uint32_t l, uint32_t old) {
    return (uint32_t)amdgcn_writelane((int)v, (int)l, (int)old);
}

// Holder value of a hash that is the same on every lane (scalar loads of
// both candidate buckets' keys and values).
__device__ inline uint32_t holder_uniform(const Table &t, uint64_t h) {
    uint32_t b1, b2;
    buckets_of(h, t.shift, t.in_block, b1, b2);
    const cptr<uint64_t> k = as_const(t.keys);
    const cptr<uint32_t> v = as_const(t.vals);
    const uint64_t k10 = k[2 * (uint64_t)b1], k11 = k[2 * (uint64_t)b1 + 1];
    const uint64_t k20 = k[2 * (uint64_t)b2], k21 = k[2 * (uint64_t)b2 + 1];
    const uint32_t v10 = v[2 * (uint64_t)b1], v11 = v[2 * (uint64_t)b1 + 1];
    const uint32_t v20 = v[2 * (uint64_t)b2], v21 = v[2 * (uint64_t)b2 + 1];
    if (h == 0) return kNoHolder;
    return k10 == h ? v10 : k11 == h ? v11 : k20 == h ? v20 : k21 == h ? v21 : kNoHolder;
}

// Lane masks of the holders of a (uniform) holder value on the C columns of
// the wavefront whose first decode is `base` (a multiple of 64 * C): the
// wavefront's words of the bitmap row (always loaded, from row 0 when the
// value is not a row, so that the load does not wait on a branch), or the
// one lane of a single holder, or none.
template <int C>
__device__ inline void holder_masks(const Table &t, uint32_t v, uint32_t base, lmask (&m)[C]) {
    const bool row = v < kHeldOne;
    const cptr<uint64_t> w = as_const(t.bits + (uint64_t)(row ? v : 0u) * t.bpitch + base / kWave);
    const uint32_t d = v & ~kHeldOne;
#pragma unroll
    for (int q = 0; q < C; ++q) {
        const uint32_t o = d - (base + (uint32_t)q * kWave);
        const lmask one = (v != kNoHolder && o < (uint32_t)kWave) ? (1ull << o) : 0ull;
        m[q] = row ? w[q] : one;
    }
}

// First-miss scan of one request's run on the columns in alive[] (the
// columns that need it), starting at block `start` (uniform, < n) whose
// holder value v0 was looked up beforehand.  Past the first block, W blocks
// are looked up per step, their holder lookups issued together.  lam[]
// holds bt * start on entry for those columns and bt * (first-miss index)
// on return (bt = tokens per block).
template <int W, int C>
__device__ inline void probe_from(const Table &t, uint32_t base, cptr<uint64_t> run, uint32_t n, uint32_t start,
                                  lmask (&alive)[C], uint32_t (&lam)[C], uint32_t bt, uint32_t v0) {
    lmask m[C];
    holder_masks<C>(t, v0, base, m);
#pragma unroll
    for (int q = 0; q < C; ++q) {
        alive[q] &= m[q];
        lam[q] += in_mask(alive[q]) ? bt : 0u;
    }
    for (uint32_t i0 = start + 1; i0 < n; i0 += W) {
        lmask any = 0;
#pragma unroll
        for (int q = 0; q < C; ++q) any |= alive[q];
        if (!any) break;
        uint32_t v[W];
#pragma unroll
        for (int w = 0; w < W; ++w) v[w] = i0 + w < n ? holder_uniform(t, run[i0 + w]) : kNoHolder;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            if (i0 + w >= n) break;
            holder_masks<C>(t, v[w], base, m);
#pragma unroll
            for (int q = 0; q < C; ++q) {
                alive[q] &= m[q];
                lam[q] += in_mask(alive[q]) ? bt : 0u;
            }
        }
    }
}

// Prefix lengths of every leader on every decode: one wavefront per
// (leader, kLeadGroups groups of 64 decodes), looping over such tasks (the
// leader count is read from device memory, so every wavefront ends after at
// most ceil(tasks / wavefronts) of them).  A task takes the leader's blocks
// 64 at a time, lane k block k: its holder value (looked up by
// lead_holder_kernel, or here when there was no room), then, per group, the
// word of its bitmap row over the group's 64 decodes (or the one-hot word of
// a single holder).  An inclusive AND across lanes, seeded with the group's
// decodes still matching, gives in lane k the decodes that hold every block
// up to k; it only loses bits as k grows, so decode l matches exactly the
// blocks below the first lane whose word lacks bit l, found by binary
// search over the words in LDS.  Writes B_tok * j for the task's decodes,
// in fp32 (exact below 2^24; only requests shorter than that read it,
// capped by their own length).
// Inclusive AND over lanes 0..l of a 32-bit value, in lane l, with DPP:
// shifts right by 1, 2, 4 and 8 within each row of 16 lanes (a lane with
// no source takes all ones), then the last lane of row 0 into row 1 and of
// row 2 into row 3, then the last lane of row 1 into rows 2 and 3.  Every
// lane must be active.
__device__ inline uint32_t wave_and_prefix_u32(uint32_t v) {
    v &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x111, 0xF, 0xF, false);   // row_shr 1
    v &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x112, 0xF, 0xF, false);   // row_shr 2
    v &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x114, 0xF, 0xF, false);   // row_shr 4
    v &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x118, 0xF, 0xF, false);   // row_shr 8
    v &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast 15
    v &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast 31
    return v;
}

__device__ inline uint64_t wave_and_prefix_u64(uint64_t v) {
    const uint32_t lo = wave_and_prefix_u32((uint32_t)v), hi = wave_and_prefix_u32((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Groups of 64 decodes per task: the task's groups share each block's
// holder value (and its load); their bitmap words load side by side.
constexpr uint32_t kLeadGroups = 2;

__global__ __launch_bounds__(kBlock) void lead_kernel(Table t, uint32_t D, uint32_t bt, const Lead *__restrict__ lead,
                                                      const unsigned int *__restrict__ n_lead, uint32_t lead_cap,
                                                      const uint32_t *__restrict__ hv,
                                                      const uint64_t *__restrict__ hashes, uint32_t ngroup,
                                                      float *__restrict__ lam_out) {
    __shared__ uint64_t pw[kWavesPerBlock][kLeadGroups][kWave];
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t wv = wave_index();
    const uint32_t nl_all = *n_lead;
    const uint32_t nl = nl_all < lead_cap ? nl_all : lead_cap;
    const uint32_t ntg = (ngroup + kLeadGroups - 1) / kLeadGroups;   // tasks per leader
    const uint64_t tasks = (uint64_t)nl * ntg;
    const uint64_t nw = (uint64_t)gridDim.x * kWavesPerBlock;
    for (uint64_t task = (uint64_t)blockIdx.x * kWavesPerBlock + wv; task < tasks; task += nw) {
        const uint32_t slot = (uint32_t)(task / ntg), g0 = (uint32_t)(task % ntg) * kLeadGroups;
        const cptr<uint32_t> w = as_const((const uint32_t *)(lead + slot));
        const uint64_t a = ((uint64_t)w[1] << 32) | (uint64_t)w[0];
        const uint64_t hoff = ((uint64_t)w[3] << 32) | (uint64_t)w[2];
        const uint32_t n = w[4], m = w[5];
        const bool pre = m != kNoPre;
        const uint32_t nb = pre ? m : n;   // blocks to take (held by someone before block m)
        // per group: the decodes (lanes) holding every block so far, and
        // this lane's decode's leading blocks held; a group past the pool
        // holds none
        uint64_t alive[kLeadGroups];
        uint32_t j[kLeadGroups];
#pragma unroll
        for (uint32_t q = 0; q < kLeadGroups; ++q) {
            alive[q] = g0 + q < ngroup ? ~0ull : 0ull;
            j[q] = 0;
        }
        auto live = [&]() {
            uint64_t x = 0;
#pragma unroll
            for (uint32_t q = 0; q < kLeadGroups; ++q) x |= alive[q];
            return x != 0;
        };
        for (uint32_t k0 = 0; k0 < nb && live(); k0 += kWave) {
            const uint32_t k = k0 + lane;
            const uint32_t nk = nb - k0 < (uint32_t)kWave ? nb - k0 : (uint32_t)kWave;
            uint32_t v = kNoHolder;
            if (k < nb) v = pre ? hv[hoff + k] : holder_lane(t, hashes[a + k]);
#pragma unroll
            for (uint32_t q = 0; q < kLeadGroups; ++q) {
                const uint32_t g = g0 + q;
                uint64_t word = 0;
                if (g < ngroup) {
                    if (v < kHeldOne) {
                        word = t.bits[(uint64_t)v * t.bpitch + g];
                    } else if (v != kNoHolder) {
                        const uint32_t o = (v & ~kHeldOne) - g * kWave;
                        word = o < (uint32_t)kWave ? 1ull << o : 0ull;
                    }
                }
                pw[wv][q][lane] = wave_and_prefix_u64(word & alive[q]);
            }
            __builtin_amdgcn_wave_barrier();
            // lane l: the number of leading words (of nk) holding bit l
#pragma unroll
            for (uint32_t q = 0; q < kLeadGroups; ++q) {
                uint32_t lo = 0, hi = nk;
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) / 2;
                    if ((pw[wv][q][mid] >> lane) & 1ull) lo = mid + 1;
                    else hi = mid;
                }
                j[q] += lo;
                alive[q] = pw[wv][q][nk - 1];
            }
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (uint32_t q = 0; q < kLeadGroups; ++q) {
            const uint32_t d = (g0 + q) * kWave + lane;
            if (g0 + q < ngroup && d < D) lam_out[(uint64_t)slot * D + d] = (float)(bt * j[q]);
        }
    }
}

// Buffer-resource word 3 for raw (untyped, unswizzled) buffer access on gfx9-class targets.
constexpr int kBufferFlags = 0x00020000;

__device__ inline float2 load_row(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t row_off) {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)row_off, 0));
}

__device__ inline uint32_t load_lam(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t row_off) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_off, (int)row_off, 0);
}

// One wavefront per (run of scoring-order requests, group of 64*C decodes);
// lane l holds decodes g*64*C + q*64 + l, q < C.  For each request of the
// run: prefix lengths min(leader's, L*), non-cached tokens, feasibility and
// cost (Eqs. (2)-(7)), then the group's K best feasible (score, index) keys
// into partial[group][position][0..K).  Token counts are below 2^24 here,
// so x = l - lambda and the feasibility test x <= xm_d are exact in fp32
// and give the costs of integer arithmetic; a request no longer than every
// limit xm_d of the group is feasible on all of them and skips the test.
// A request marked in its record (its leader did not fit the leader table,
// or it has 2^24 tokens or more) is matched from block 0 on its own and
// scored in integers.  Requests of one prefill are consecutive, so the
// snapshot row stays in registers and is reloaded only when the prefill
// changes; the leader's prefix lengths are kept too, and the next
// request's are fetched during the current step only when its leader row
// differs.  Records are read two requests ahead.  Requests are taken in
// chunks of 64/K whose keys are gathered one per lane and stored together.
// The cost of a pair with x non-cached tokens from its derived row(s), as
// fp32 bits: the direct route, or the cheaper of the direct and the staged
// route (costs are non-negative, so the smaller bits are the smaller cost;
// ties keep the direct route's value, which is the same).
template <bool TWO>
__device__ inline uint32_t route_cost(float x, float2 r1, float2 r2) {
    const uint32_t c1 = __float_as_uint(fmaf(x, r1.x, r1.y));
    if (!TWO) return c1;
    return min(c1, __float_as_uint(fmaf(x, r2.x, r2.y)));
}

// Merged mode (MERGE, at most kMaxMergeGroups groups; used for a pool of
// one group, where it saves the merge kernel): a workgroup is one run,
// its wavefront w the decode group w; at the end of each chunk of requests
// the wavefronts put their top-k keys in LDS (two buffers, alternating by
// chunk), and after one barrier each wavefront merges a share of the
// chunk's requests over all groups and writes their outputs.  A buffer is
// written again only two chunks later, after the next barrier, which every
// wavefront reaches only once its merge of the buffer is done.  Workgroups
// go to the XCDs in turn, and XCD x takes the x-th contiguous eighth of the
// runs, so its L2 holds the snapshot rows of its own prefills.
constexpr uint32_t kMaxMergeGroups = 8;

// Without per-pair outputs the kernel is held to 80 registers, so that a
// SIMD keeps 6 wavefronts (the staged-route variant needs one register
// more than that when left alone).
template <int K, int W, int C, bool PAIRS, bool TWO, bool MERGE>
__global__ __launch_bounds__(MERGE ? kWave * kMaxMergeGroups : kBlock, PAIRS ? 1 : 6)
void score_kernel(Snap s, Table t, const Hot *__restrict__ hot, const Cold *__restrict__ cold,
                  const float *__restrict__ lead_lam, uint32_t lead_rows, const uint64_t *__restrict__ hashes,
                  const uint32_t *__restrict__ len_tokens, const uint64_t *__restrict__ hash_off,
                  const uint32_t *__restrict__ n_valid, uint32_t n_req, uint32_t run_len, uint32_t n_runs,
                  uint32_t ngroup, uint64_t *__restrict__ partial, PairOut po, uint32_t k_out,
                  int32_t *__restrict__ out_idx, float *__restrict__ out_score) {
    __shared__ uint64_t mkeys[MERGE ? 2 : 1][MERGE ? kMaxMergeGroups : 1][kWave];
    const uint32_t lane = threadIdx.x % kWave;
    uint32_t run, grp;
    if (MERGE) {
        const uint32_t rpx = (n_runs + kXcds - 1) / kXcds;
        run = (blockIdx.x % kXcds) * rpx + blockIdx.x / kXcds;
        grp = wave_index();
    } else if (ngroup % kXcds == 0) {
        // workgroups go to the XCDs in turn: XCD x takes groups
        // [x*gx, (x+1)*gx), so its decodes' snapshot columns stay in its
        // own L2; the waves of a workgroup take consecutive runs of one group
        const uint32_t gx = ngroup / kXcds, x = blockIdx.x % kXcds, k = blockIdx.x / kXcds;
        grp = x * gx + k % gx;
        run = (k / gx) * kWavesPerBlock + wave_index();
    } else {
        const uint32_t gw = blockIdx.x * kWavesPerBlock + wave_index();
        run = gw / ngroup;
        grp = gw % ngroup;
    }
    if (run >= n_runs) return;
    const uint32_t nv = *n_valid;
    const uint32_t i0 = run * run_len;
    if (i0 >= nv) return;
    const uint32_t i1 = (i0 + run_len < nv) ? i0 + run_len : nv;
    const uint32_t base = grp * (kWave * C);
    const uint32_t bt = s.block_tokens;
    uint32_t d[C];
    float xmf[C];
    bool act[C];
    // x = l - lambda is feasible iff x < xlim, i.e. x <= xlim - 1 for
    // xlim >= 1; xlim = 0 never is (limit -1).  Limits above 2^24 are taken
    // as 2^24, which every x scored in fp32 is below.  A column past the
    // pool has limit NaN, which no x passes, whatever its loads read.  xlo:
    // the least limit of the lane's decodes as fp32 bits, 0 when one is
    // never feasible (so a group with columns past the pool, and requests
    // of at least one token, never take the all-feasible path).
    uint32_t xlo = 0xFFFFFFFFu;
#pragma unroll
    for (int q = 0; q < C; ++q) {
        d[q] = base + q * kWave + lane;
        act[q] = d[q] < s.D;
        const uint64_t xlim = act[q] ? s.dxlim[d[q]] : 0;
        xmf[q] = !act[q] ? __builtin_nanf("")
                 : xlim == 0 ? -1.0f
                             : (float)(xlim - 1 < kExactTok ? xlim - 1 : (uint64_t)kExactTok);
        xlo = min(xlo, xlim == 0 ? 0u : __float_as_uint(xmf[q]));
    }
    // column q of the lane is at lane offset (base + lane + 64 q) * size;
    // the 64 q part is a constant that the loads carry in their offset
    // field, so the lane needs one offset register per table.  Columns past
    // the pool read what follows the last decode: the next row, or the
    // kRowPad elements allocated after the last row.
    constexpr uint32_t kRowStep = kWave * (uint32_t)sizeof(float2), kLamStep = kWave * (uint32_t)sizeof(float);
    const uint32_t voff = (base + lane) * (uint32_t)sizeof(float2);
    const uint32_t loff = (base + lane) * (uint32_t)sizeof(float);
    // a request of at most xall tokens (fp32 bits) is feasible on every
    // decode of the group
    const uint32_t xall = wave_min_u32_dpp(xlo);
    const cptr<uint64_t> chash = as_const(hashes);
    // rows of (seconds per token, constant part) and the leaders' prefix
    // lengths through buffer resources: a row's byte offset is the scalar
    // offset, the column's the lane offset
    const uint64_t sl_bytes = ((uint64_t)s.P * s.slp + kRowPad) * sizeof(float2);   // < 2^32 (checked at load)
    const uint64_t ll_bytes = ((uint64_t)lead_rows * s.D + kRowPad) * sizeof(float);   // < 2^32 (capped)
    const __amdgpu_buffer_rsrc_t slr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)s.sl, (short)0, (int)(uint32_t)(sl_bytes < 0xFFFFFFFFull ? sl_bytes : 0xFFFFFFFFull), kBufferFlags);
    const __amdgpu_buffer_rsrc_t llr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)lead_lam, (short)0, (int)(uint32_t)(ll_bytes < 0xFFFFFFFFull ? ll_bytes : 0xFFFFFFFFull),
        kBufferFlags);
    const __amdgpu_buffer_rsrc_t srr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(TWO ? s.sr : s.sl), (short)0,
        (int)(uint32_t)(sl_bytes < 0xFFFFFFFFull ? sl_bytes : 0xFFFFFFFFull), kBufferFlags);
    Hot c0 = load_hot(hot, i0);
    Hot c1 = load_hot(hot, i0 + 1);
    float2 rowv[C], rowv2[C];   // the current prefill's row (and its staged-route row)
    uint32_t rowcur = c0.row;
    // the current leader's B_tok * j (the next one's while it loads), as
    // fp32 bits: non-negative, so their order is that of the unsigned bits
    uint32_t laml[C];
#pragma unroll
    for (int q = 0; q < C; ++q) {
        rowv[q] = load_row(slr, voff + q * kRowStep, c0.row);
        rowv2[q] = TWO ? load_row(srr, voff + q * kRowStep, c0.row) : rowv[q];
        laml[q] = load_lam(llr, loff + q * kLamStep, c0.lrow);
    }
    constexpr uint32_t kPer = kWave / K;   // requests whose keys one store writes
    uint32_t pc_bits = 0xFFFFFFFFu, pc_idx = 0xFFFFFFFFu;   // gathered keys (empty = ~0)

    // one request's column costs (fp32 bits, ~0 where infeasible):
    // scoring-order position i, its record and the next one's (whose leader
    // values are fetched while i is scored)
    auto cost = [&](uint32_t i, const Hot &cur, const Hot &nxt, Hot &ahead, uint32_t (&cb)[C]) {
        // the lane offsets of the loads below are tied to the request (an
        // empty asm, no instruction) so that each column's offset stays in
        // the load's offset field instead of a register of its own
        if (cur.row != rowcur) {
            uint32_t vo = voff;
            asm("" : "+v"(vo) : "s"(i));
#pragma unroll
            for (int q = 0; q < C; ++q) {
                rowv[q] = load_row(slr, vo + q * kRowStep, cur.row);
                if (TWO) rowv2[q] = load_row(srr, vo + q * kRowStep, cur.row);
            }
            rowcur = cur.row;
        }
        // the record two ahead, issued after the last use of the loaded
        // records' fields (scalar loads complete out of order, so a use
        // after it would wait for it)
        __builtin_amdgcn_sched_barrier(0);
        ahead = load_hot(hot, i + 2);
        uint32_t r_out = 0;
        if (PAIRS) r_out = load_cold(cold, i).r;
        // this request's prefix lengths B_tok * j (fp32 bits): its leader's,
        // capped by its own common run with the leader; then the next
        // request's leader values, if its leader row differs, are loaded
        // over the current ones, whose last use this is (with staged routes,
        // after the costs: there the kernel has no registers for both sets
        // beside the costs' operands)
        uint32_t lam[C];
#pragma unroll
        for (int q = 0; q < C; ++q) lam[q] = min(laml[q], cur.lams);
        auto reload = [&]() {
            if (nxt.lrow != cur.lrow) {
                uint32_t lo = loff;
                asm("" : "+v"(lo) : "s"(i));
#pragma unroll
                for (int q = 0; q < C; ++q) laml[q] = load_lam(llr, lo + q * kLamStep, nxt.lrow);
            }
        };
        if (!TWO) reload();
        if ((int32_t)cur.lams < 0) {
            // matched on its own from block 0, in integers (exact)
            const uint32_t r = load_cold(cold, i).r;
            const uint32_t len = as_const(len_tokens)[r];
            const uint64_t ha = as_const(hash_off)[r];
            const uint32_t hn = (uint32_t)(as_const(hash_off)[r + 1] - ha);
            lmask alive[C];
            uint32_t lam[C];
#pragma unroll
            for (int q = 0; q < C; ++q) {
                lam[q] = 0;
                alive[q] = ~0ull;
            }
            if (hn)
                probe_from<W, C>(t, base, chash + ha, hn, 0, alive, lam, bt, holder_uniform(t, chash[ha]));
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const uint32_t x = len - lam[q];
                const uint64_t xlim = act[q] ? s.dxlim[d[q]] : 0;
                const bool feas = (uint64_t)x < xlim;
                const float cost = __uint_as_float(route_cost<TWO>((float)x, rowv[q], rowv2[q]));
                if (PAIRS && act[q]) {
                    const uint64_t o = (uint64_t)r_out * s.D + d[q];
                    const uint32_t jq = lam[q] / bt;
                    if (po.j) po.j[o] = (uint16_t)(jq < 0xFFFFu ? jq : 0xFFFFu);
                    if (po.feas) po.feas[o] = feas ? 1 : 0;
                    if (po.score) po.score[o] = cost;
                }
                cb[q] = feas ? __float_as_uint(cost) : 0xFFFFFFFFu;
            }
        } else {
            // non-cached tokens (Eq. (2) / bpt), feasibility and the cost of Eq. (5)
            const float lenf = __uint_as_float(cur.len);
            if (!PAIRS && cur.len <= xall) {
#pragma unroll
                for (int q = 0; q < C; ++q)
                    cb[q] = route_cost<TWO>(lenf - __uint_as_float(lam[q]), rowv[q], rowv2[q]);
            } else {
#pragma unroll
                for (int q = 0; q < C; ++q) {
                    const float x = lenf - __uint_as_float(lam[q]);
                    const bool feas = x <= xmf[q];
                    const float cost = __uint_as_float(route_cost<TWO>(x, rowv[q], rowv2[q]));
                    if (PAIRS && act[q]) {
                        const uint64_t o = (uint64_t)r_out * s.D + d[q];
                        const uint32_t jq = (uint32_t)__uint_as_float(lam[q]) / bt;
                        if (po.j) po.j[o] = (uint16_t)(jq < 0xFFFFu ? jq : 0xFFFFu);
                        if (po.feas) po.feas[o] = feas ? 1 : 0;
                        if (po.score) po.score[o] = cost;
                    }
                    cb[q] = feas ? __float_as_uint(cost) : 0xFFFFFFFFu;
                }
            }
        }
        if (TWO) reload();
    };
    auto lane_min = [&](const uint32_t (&cb)[C]) {
        uint32_t lm = cb[0];
#pragma unroll
        for (int q = 1; q < C; ++q) lm = min(lm, cb[q]);
        return lm;
    };
    // one of the group's best, of cost bits mn (uniform; ~0 when no
    // feasible candidate is left, and nothing is kept): the least decode
    // index holding it, i.e. the lowest lane holding it in the first column
    // that holds it, whose cost is then removed; its key goes to lane e
    auto place = [&](uint32_t e, uint32_t mn, uint32_t (&cb)[C], bool more) {
        if (mn == 0xFFFFFFFFu) return false;
        uint32_t dm = 0;
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const lmask m = ballot(cb[q] == mn);
            if (m) {
                const uint32_t l = (uint32_t)__builtin_ctzll(m);
                dm = base + q * kWave + l;
                if (more && lane == l) cb[q] = 0xFFFFFFFFu;
                break;
            }
        }
        pc_bits = write_lane(mn, e, pc_bits);
        pc_idx = write_lane(dm, e, pc_idx);
        return true;
    };
    // one request scored and its K best kept: least cost bits, then least
    // decode index
    auto step = [&](uint32_t i, uint32_t g0, const Hot &cur, const Hot &nxt, Hot &ahead) {
        uint32_t cb[C];
        cost(i, cur, nxt, ahead, cb);
        const uint32_t slot = i - g0;
#pragma unroll
        for (int r = 0; r < K; ++r)
            if (!place(slot * K + (uint32_t)r, wave_min_u32_dpp(lane_min(cb)), cb, r + 1 < K)) break;
    };

    for (uint32_t g0 = i0; g0 < i1; g0 += kPer) {
        const uint32_t g1 = (g0 + kPer < i1) ? g0 + kPer : i1;
        uint32_t i = g0;
        // three requests per trip: each record is loaded into the registers
        // of the one whose step has just ended, so the records rotate
        // without copies; for K = 1 the three requests' minima are taken
        // together (not with per-pair outputs or staged routes, whose
        // variants would then need more registers than 6 wavefronts per
        // SIMD leave)
        for (; i + 3 <= g1; i += 3) {
            Hot c2, c3, c4;
            if (K == 1 && !PAIRS && !TWO) {
                uint32_t ca[C], cb[C], cc[C];
                cost(i, c0, c1, c2, ca);
                cost(i + 1, c1, c2, c3, cb);
                cost(i + 2, c2, c3, c4, cc);
                uint32_t ma, mb, mc;
                wave_min3_u32(lane_min(ca), lane_min(cb), lane_min(cc), ma, mb, mc);
                place(i - g0, ma, ca, false);
                place(i + 1 - g0, mb, cb, false);
                place(i + 2 - g0, mc, cc, false);
            } else {
                step(i, g0, c0, c1, c2);
                step(i + 1, g0, c1, c2, c3);
                step(i + 2, g0, c2, c3, c4);
            }
            c0 = c3;
            c1 = c4;
        }
        for (; i < g1; ++i) {
            Hot c2;
            step(i, g0, c0, c1, c2);
            c0 = c1;
            c1 = c2;
        }
        const uint64_t key = ((uint64_t)pc_bits << 32) | (uint64_t)pc_idx;
        if (MERGE) {
            const uint32_t buf = ((g0 - i0) / kPer) & 1u;
            mkeys[buf][grp][lane] = key;
            __syncthreads();
            // request slot sl of the chunk (its keys in lanes sl*K ..
            // sl*K+K-1 of every group) is merged by lane sl / ngroup of
            // wavefront sl % ngroup
            const uint32_t sl = grp + lane * ngroup;
            if (sl < g1 - g0) {
                uint64_t best[K];
#pragma unroll
                for (int q = 0; q < K; ++q) best[q] = kEmptyKey;
                for (uint32_t g = 0; g < ngroup; ++g) {
#pragma unroll
                    for (int q = 0; q < K; ++q) {
                        const uint64_t x = mkeys[buf][g][sl * K + q];
                        if (x < best[K - 1]) topk_insert<K>(best, x);
                    }
                }
                const uint64_t o = (uint64_t)cold[g0 + sl].r * k_out;
                for (uint32_t q = 0; q < k_out; ++q) {
                    const uint64_t m = best[q];
                    out_idx[o + q] = m == kEmptyKey ? -1 : (int32_t)(uint32_t)m;
                    out_score[o + q] = m == kEmptyKey ? __builtin_inff() : __uint_as_float((uint32_t)(m >> 32));
                }
            }
        } else if (lane < (g1 - g0) * K) {
            // the lane tied to the chunk (an empty asm, no instruction), so
            // that the store's address is formed here instead of held in
            // registers through the loop
            uint32_t ln = lane;
            asm("" : "+v"(ln) : "s"(g0));
            partial[((uint64_t)grp * n_req + g0) * K + ln] = key;
        }
        pc_bits = 0xFFFFFFFFu;
        pc_idx = 0xFFFFFFFFu;
    }
}

// Merge the per-group keys of every scoring-order request into its top-k
// (ascending (score, index)) and write it at the request's own position;
// invalid requests (ordered last) get index -1 and score NaN.
template <int K>
__global__ __launch_bounds__(256) void reduce_kernel(uint32_t n_req, uint32_t nchunk, uint32_t k,
                                                     const uint64_t *__restrict__ partial,
                                                     const Cold *__restrict__ cold,
                                                     const uint32_t *__restrict__ n_valid,
                                                     int32_t *__restrict__ out_idx, float *__restrict__ out_score) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_req) return;
    const uint64_t o = (uint64_t)cold[i].r * k;
    if (i >= *n_valid) {
        for (uint32_t q = 0; q < k; ++q) {
            out_idx[o + q] = -1;
            out_score[o + q] = __builtin_nanf("");
        }
        return;
    }
    uint64_t best[K];
#pragma unroll
    for (int q = 0; q < K; ++q) best[q] = kEmptyKey;
    for (uint32_t c = 0; c < nchunk; ++c) {
        const uint64_t *src = partial + ((uint64_t)c * n_req + i) * K;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const uint64_t x = src[q];
            if (x < best[K - 1]) topk_insert<K>(best, x);
        }
    }
#pragma unroll
    for (int q = 0; q < K; ++q) {
        if ((uint32_t)q < k) {
            const uint64_t m = best[q];
            out_idx[o + q] = m == kEmptyKey ? -1 : (int32_t)(uint32_t)m;
            out_score[o + q] = m == kEmptyKey ? __builtin_inff() : __uint_as_float((uint32_t)(m >> 32));
        }
    }
}

// Orders one wavefront's LDS accesses around an exchange between its lanes
// (its LDS operations execute in order, so it costs no instruction).
__device__ inline void lane_phase() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Leading 64-bit words of the 64 in LDS (each the AND of those before it, low
// and high halves in turn) that have the lane's bit, 0 .. 64.
__device__ inline uint32_t count_words(const uint32_t *wds, uint32_t lane) {
    const uint32_t *half = wds + (lane >> 5);
    const uint32_t sh = lane & 31u;
    uint32_t j = 0;
#pragma unroll
    for (uint32_t b = 32; b; b >>= 1) j += (half[2 * (j + b - 1)] >> sh & 1u) * b;
    return j + (half[2 * j] >> sh & 1u);   // 63 found so far: the last word
}

// Holder values of two hashes, the loads of both together (hash 0: none).
__device__ inline void holder_lane2(const Table &t, const uint64_t (&h)[2], uint32_t (&v)[2]) {
    uint64_t slot[2];
    ulonglong2 k1[2], k2[2];
    uint32_t b1[2], b2[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        buckets_of(h[u], t.shift, t.in_block, b1[u], b2[u]);
        k1[u] = *(const ulonglong2 *)(t.keys + 2 * (uint64_t)b1[u]);
        k2[u] = *(const ulonglong2 *)(t.keys + 2 * (uint64_t)b2[u]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const uint64_t x = h[u];
        slot[u] = x == 0 ? ~0ull
                : k1[u].x == x ? 2 * (uint64_t)b1[u] : k1[u].y == x ? 2 * (uint64_t)b1[u] + 1
                : k2[u].x == x ? 2 * (uint64_t)b2[u] : k2[u].y == x ? 2 * (uint64_t)b2[u] + 1 : ~0ull;
        v[u] = kNoHolder;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (slot[u] != ~0ull) v[u] = t.vals[slot[u]];
}

// ---------------------------------------------------------------- direct selection
//
// Small batches in one launch, with no ordering: the ordering pipeline is 10
// to 25 launches of 3-10 us each, while the matching it saves (one scan per
// shared prefix instead of one per request) costs a small batch less than
// that.  One wavefront per request (or `nw` of them, each a share of the
// decodes): lanes look up the holder values of 64 blocks at a time, up to the
// first block no decode holds; then, per chunk of C groups of 64 decodes, the
// blocks' bitmap words are ANDed block by block (scalar), each decode lane
// counting the blocks it still matches.  Runs with more than 64 held blocks go
// 128 at a time: a lane loads its blocks' words, the ANDs go over the lanes
// and each decode lane finds its count by a binary search (a run of 4,096 held
// blocks on 48 / 768 decodes 364 / 778 us block by block, 54 / 98 so;
// the ordering pipeline 178 / 186).  Costs, feasibility and the top-k
// are those of the scoring kernel bit for bit: x < 2^24 is the same integer
// in fp32 and in u32, and larger x are rounded to fp32 as there.  fly: the
// cost factors are computed here from the snapshot instead of read from the
// derived rows (saves derive_kernel's launch).  With hotr, each request's
// record and its row of B_tok * j are written for the ranking sweep, every
// request being its own leader (row r of lam).
template <int K, int C>
__global__ __launch_bounds__(kBlock) void direct_kernel(Snap s, Table t, Reqs rq, uint32_t nw, bool fly,
                                                        uint32_t k_out, int32_t *__restrict__ out_idx,
                                                        float *__restrict__ out_score, uint32_t *__restrict__ err,
                                                        Hot *__restrict__ hotr, float *__restrict__ lam) {
    constexpr int G = C < 4 ? C : 4;   // columns whose words are exchanged together
    __shared__ uint64_t wkeys[kWavesPerBlock][K];
    __shared__ __align__(8) uint32_t wds[kWavesPerBlock][2][G][2 * kWave];
    const uint32_t lane = threadIdx.x % kWave, wv = wave_index();
    const uint32_t r = blockIdx.x * (kWavesPerBlock / nw) + wv / nw, part = wv % nw;
    if (r >= rq.n_req) return;   // only with one wavefront per request (no barrier then)
    const uint32_t p = as_const(rq.prefill)[r], len = as_const(rq.len)[r];
    const uint64_t a = as_const(rq.off)[r], b = as_const(rq.off)[r + 1];
    const bool ok = p < s.P && len >= 1 && b >= a && b <= rq.n_hashes && b - a == (uint64_t)(len / s.block_tokens);
    uint64_t best[K];
#pragma unroll
    for (int q = 0; q < K; ++q) best[q] = kEmptyKey;
    if (ok) {
        const uint32_t n = (uint32_t)(b - a), bt = s.block_tokens;
        // holder values of blocks k0 .. k0+63, one per lane; returns how many
        // blocks from k0 on some decode holds
        auto lookup = [&](uint32_t k0, uint32_t &v) {
            const uint32_t k = k0 + lane;
            v = k < n ? holder_lane(t, rq.hashes[a + k]) : kNoHolder;
            const lmask none = ballot(v == kNoHolder);
            return none ? (uint32_t)__builtin_ctzll(none) : (uint32_t)kWave;
        };
        uint32_t v0 = kNoHolder;
        const uint32_t m0 = lookup(0, v0);   // n = 0 gives 0
        for (uint32_t base = part * kWave * C; base < s.D; base += nw * kWave * C) {
            // this lane's leading blocks on each column's decode
            lmask alive[C];
            uint32_t j[C];
#pragma unroll
            for (int q = 0; q < C; ++q) {
                alive[q] = ~0ull;
                j[q] = 0;
            }
            if (m0 < (uint32_t)kWave || n <= (uint32_t)kWave) {
                constexpr uint32_t U = C > 4 ? 2 : 4;   // blocks whose words load together
                lmask any = ~0ull;
                for (uint32_t k = 0; k < m0 && any; k += U) {
                    lmask w[U][C];
#pragma unroll
                    for (uint32_t u = 0; u < U; ++u) {
                        const uint32_t vk = k + u < m0 ? (uint32_t)__builtin_amdgcn_readlane((int)v0, (int)((k + u) % kWave))
                                                       : kNoHolder;
                        holder_masks<C>(t, vk, base, w[u]);
                    }
                    any = 0;
#pragma unroll
                    for (uint32_t u = 0; u < U; ++u) {
#pragma unroll
                        for (int q = 0; q < C; ++q) {
                            alive[q] &= w[u][q];
                            j[q] += in_mask(alive[q]) ? 1u : 0u;
                        }
                    }
#pragma unroll
                    for (int q = 0; q < C; ++q) any |= alive[q];
                }
            } else {
                for (uint32_t k0 = 0;; k0 += 2 * kWave) {
                    uint64_t hs[2];
                    uint32_t v[2];
#pragma unroll
                    for (uint32_t u = 0; u < 2; ++u) {
                        const uint32_t k = k0 + u * kWave + lane;
                        hs[u] = k < n ? rq.hashes[a + k] : 0ull;
                    }
                    holder_lane2(t, hs, v);
                    const lmask none0 = ballot(v[0] == kNoHolder), none1 = ballot(v[1] == kNoHolder);
                    lmask any = 0;
#pragma unroll
                    for (int q0 = 0; q0 < C; q0 += G) {
                        lmask w[2][G];
#pragma unroll
                        for (uint32_t u = 0; u < 2; ++u) {
                            const bool row = v[u] < kHeldOne;
                            const uint64_t *src = t.bits + (uint64_t)(row ? v[u] : 0u) * t.bpitch + base / kWave + q0;
#pragma unroll
                            for (int q = 0; q < G; ++q) w[u][q] = src[q];
                            const uint32_t d = v[u] & ~kHeldOne;
#pragma unroll
                            for (int q = 0; q < G; ++q) {
                                const uint32_t o = d - (base + (uint32_t)(q0 + q) * kWave);
                                if (!row) w[u][q] = v[u] != kNoHolder && o < (uint32_t)kWave ? 1ull << o : 0ull;
                                w[u][q] = wave_and_prefix_u64(w[u][q] & alive[q0 + q]);
                            }
                        }
                        lane_phase();
#pragma unroll
                        for (uint32_t u = 0; u < 2; ++u) {
#pragma unroll
                            for (int q = 0; q < G; ++q) {
                                wds[wv][u][q][2 * lane] = (uint32_t)w[u][q];
                                wds[wv][u][q][2 * lane + 1] = (uint32_t)(w[u][q] >> 32);
                            }
                        }
                        lane_phase();
#pragma unroll
                        for (int q = 0; q < G; ++q) {
                            const uint32_t c0 = count_words(wds[wv][0][q], lane), c1 = count_words(wds[wv][1][q], lane);
                            j[q0 + q] += c0 + (c0 == (uint32_t)kWave ? c1 : 0u);
                            alive[q0 + q] = ballot(c0 == (uint32_t)kWave && c1 == (uint32_t)kWave);
                            any |= alive[q0 + q];
                        }
                        lane_phase();
                    }
                    // (a block that no decode holds, the run's end among them, leaves none)
                    if (none0 || none1 || !any) break;
                }
            }
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const uint32_t d = base + q * kWave + lane;
                if (d < s.D) {
                    const uint32_t x = len - bt * j[q];
                    float cost;
                    bool feas;
                    if (fly) {
                        const uint64_t pd = (uint64_t)p * s.D + d;
                        const uint32_t tau = s.tier_map[pd] & 3u;
                        cost = fmaf((float)x, sec_per_token(s, tau, p, s.util[pd]),
                                    __fadd_rn(tier_latency(s, tau), load_term(s, d)));
                        // bpt x <= m_d - m_min, both below 2^64
                        const uint64_t mem = s.free_mem[d];
                        feas = mem >= s.m_min && (uint64_t)s.bpt * x <= mem - s.m_min;
                    } else {
                        const uint64_t o = (uint64_t)p * s.slp + d;
                        const float2 r1 = s.sl[o];
                        uint32_t cb = __float_as_uint(fmaf((float)x, r1.x, r1.y));
                        if (s.sr) {
                            const float2 r2 = s.sr[o];
                            cb = min(cb, __float_as_uint(fmaf((float)x, r2.x, r2.y)));
                        }
                        cost = __uint_as_float(cb);
                        feas = (uint64_t)x < s.dxlim[d];
                    }
                    if (hotr) lam[(uint64_t)r * s.D + d] = (float)(bt * j[q]);
                    const uint64_t key = feas ? ((uint64_t)__float_as_uint(cost) << 32) | d : kEmptyKey;
                    if (key < best[K - 1]) topk_insert<K>(best, key);
                }
            }
        }
    }
    if (hotr && part == 0 && lane == 0) {
        const bool own = len >= kExactTok;
        hotr[r] = ok ? Hot{p * s.slp * (uint32_t)sizeof(float2), own ? 0u : r * s.D * (uint32_t)sizeof(float),
                           __float_as_uint((float)len), __float_as_uint(own ? -1.0f : __builtin_inff())}
                     : Hot{0, 0, 0, 0};
    }
    // the wavefront's K least keys, in lanes 0 .. K-1
    uint64_t mine = kEmptyKey;
    auto wave_best = [&](uint64_t head, uint64_t &mn) {
        const uint32_t hi = wave_min_u32_dpp((uint32_t)(head >> 32));
        const uint32_t lo = wave_min_u32_dpp((uint32_t)(head >> 32) == hi ? (uint32_t)head : 0xFFFFFFFFu);
        mn = ((uint64_t)hi << 32) | lo;
    };
#pragma unroll
    for (int q = 0; q < K; ++q) {
        uint64_t mn;
        wave_best(best[0], mn);
        if (lane == (uint32_t)q) mine = mn;
        if (q + 1 < K && best[0] == mn) {   // keys differ, so one lane pops (or all do when nothing is left)
#pragma unroll
            for (int u = 0; u + 1 < K; ++u) best[u] = best[u + 1];
            best[K - 1] = kEmptyKey;
        }
    }
    if (nw > 1) {   // one request per workgroup: every wavefront arrives here
        if (lane < (uint32_t)K) wkeys[wv][lane] = mine;
        __syncthreads();
        if (part != 0) return;
        uint64_t head = lane < nw * K ? wkeys[lane / K][lane % K] : kEmptyKey;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            uint64_t mn;
            wave_best(head, mn);
            if (lane == (uint32_t)q) mine = mn;
            if (head == mn) head = kEmptyKey;
        }
    }
    if (lane < k_out) {
        const uint64_t o = (uint64_t)r * k_out + lane;
        out_idx[o] = !ok || mine == kEmptyKey ? -1 : (int32_t)(uint32_t)mine;
        out_score[o] = !ok ? __builtin_nanf("") : mine == kEmptyKey ? __builtin_inff()
                                                                    : __uint_as_float((uint32_t)(mine >> 32));
    }
    if (!ok && part == 0 && lane == 0) atomicOr(err, kErrRequest);
}

// ---------------------------------------------------------------- bounded selection
//
// Batches beyond the direct selection, without ordering: on most snapshots most
// (request, decode) pairs cannot win, and a bound per group of 64 decodes shows it.
// With x >= xlo non-cached tokens on every decode of group g,
//     cost >= fma(xlo, least spt of the group, least constant of the group),
// in fp32 as well, since each operand is no larger and rounding is monotone.
// xlo = l - B_tok * m, m = leading blocks that any decode holds.  A request
// is scored on the group of least bound; every other group whose bound
// exceeds the K-th best cost so far is ruled out, and the rest are scored
// too, so the selection is the exact top-k with its ties.  Network tiers
// differ by factors, so on fat trees 1.1 of 48 groups are scored on average
// (2 to 4 for k = 3 under memory pressure).
//   derive_bound_kernel -- the cost factors, and per (p, group) the bound's.
//   match_kernel        -- per request the holder values of its leading held
//                          blocks and their count m.
//   bounded_kernel      -- bounds, scoring, top-k, outputs.
// Where little can be ruled out every group is scored by one wavefront,
// which costs more than the ordering pipeline's shared scans: spread_kernel
// measures how many groups a snapshot's bounds leave when it is loaded.

// lanes per request of match_kernel, and blocks per lane and step (measured at
// 1,048,576 requests of 25 blocks / 262,144 of 191 / 99,991 of 25, us: 16 x 2
// 303 / 261 / 29, 8 x 2 250 / 266 / 30, 8 x 4 265 / 264 / 30, 4 x 4 236 / 279 /
// 40, 4 x 8 301 / 278 / 38)
constexpr uint32_t kStepLanes = 8, kStepBlocks = 2;
constexpr uint32_t kBoundMaxGroups = kWave;   // one lane per group: pools of up to 4,096 decodes

struct Bounds {
    const float2 *lo;    // [P][ngroup] least spt and constant of the group
    const float2 *lo2;   // the staged routes', or null
    const float *xm;     // [ngroup * 64] largest feasible x of a decode, capped at 2^24; -1: none
    const float *xg;     // [ngroup] the group's largest xm
    uint32_t ngroup;
};

// Least value over the wavefront of four registers at once, in a .. d of
// every lane (the scheme of wave_min3_u32 with the fourth value in the rows
// it leaves unused).
__device__ inline void wave_min4_u32(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&m)[4]) {
    const auto s1 = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    const auto s2 = __builtin_amdgcn_permlane32_swap(c, d, false, false);
    const uint32_t x = min((uint32_t)s1[0], (uint32_t)s1[1]), y = min((uint32_t)s2[0], (uint32_t)s2[1]);
    const auto s16 = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    uint32_t z = min((uint32_t)s16[0], (uint32_t)s16[1]);
    z = min(z, dpp_u32<0xB1>(z));
    z = min(z, dpp_u32<0x4E>(z));
    z = min(z, dpp_u32<0x124>(z));
    z = min(z, dpp_u32<0x128>(z));
    m[0] = (uint32_t)__builtin_amdgcn_readlane((int)z, 0);
    m[1] = (uint32_t)__builtin_amdgcn_readlane((int)z, 32);
    m[2] = (uint32_t)__builtin_amdgcn_readlane((int)z, 16);
    m[3] = (uint32_t)__builtin_amdgcn_readlane((int)z, 48);
}

// One wavefront per (p, group of 64 decodes): the derived row entries and the
// bound's factors; p = 0's wavefronts also write the per-decode values.
__global__ __launch_bounds__(kBlock) void derive_bound_kernel(Snap s, const uint8_t *__restrict__ t1,
                                                              const float *__restrict__ u1,
                                                              const uint8_t *__restrict__ t2,
                                                              const float *__restrict__ u2, uint32_t ngroup,
                                                              float2 *__restrict__ sl, float2 *__restrict__ sr,
                                                              float *__restrict__ dbase, uint64_t *__restrict__ dxlim,
                                                              float2 *__restrict__ lo, float2 *__restrict__ lo2,
                                                              float *__restrict__ xm, float *__restrict__ xg) {
    const uint32_t lane = threadIdx.x % kWave;
    const uint64_t task = (uint64_t)blockIdx.x * kWavesPerBlock + wave_index();
    const uint32_t p = (uint32_t)(task / ngroup), g = (uint32_t)(task % ngroup), d = g * kWave + lane;
    if (p >= s.P) return;
    const bool in = d < s.D;
    // least values as fp32 bits (non-negative); a staged route's likewise
    float2 a = make_float2(__builtin_inff(), __builtin_inff()), b = a;
    const float base = in ? load_term(s, d) : 0.0f;
    if (in) {
        const uint64_t i = (uint64_t)p * s.D + d;
        const uint32_t tau = s.tier_map[i] & 3u;
        a = make_float2(sec_per_token(s, tau, p, s.util[i]), __fadd_rn(tier_latency(s, tau), base));
        sl[(uint64_t)p * s.slp + d] = a;
        if (sr) {
            const uint32_t x = t1[i] & 3u, y = t2[i] & 3u;
            b = make_float2(sec_per_token(s, x, p, u1[i]) + sec_per_token_n(s, y, 0.0f, u2[i]),
                            __fadd_rn(__fadd_rn(tier_latency(s, x), tier_latency(s, y)), base));
            sr[(uint64_t)p * s.slp + d] = b;
        }
    }
    uint32_t m[4];
    wave_min4_u32(__float_as_uint(a.x), __float_as_uint(a.y), __float_as_uint(b.x), __float_as_uint(b.y), m);
    // a finite factor, so that xlo = 0 gives the constant and not NaN
    const uint32_t top = 0x7F7FFFFFu;
    if (lane == 0) {
        lo[task] = make_float2(__uint_as_float(min(m[0], top)), __uint_as_float(m[1]));
        if (sr) lo2[task] = make_float2(__uint_as_float(min(m[2], top)), __uint_as_float(m[3]));
    }
    if (p == 0) {
        const uint64_t lim = in ? feasible_limit(s, s.free_mem[d]) : 0;
        // largest feasible x plus one, at most 2^24 + 1
        const uint32_t x1 = (uint32_t)(lim <= kExactTok ? lim : (uint64_t)kExactTok + 1);
        xm[d] = (float)((int32_t)x1 - 1);
        if (in) {
            dbase[d] = base;
            dxlim[d] = lim;
        }
        const uint32_t most = kExactTok + 1u - wave_min_u32_dpp(kExactTok + 1u - x1);
        if (lane == 0) xg[g] = (float)((int32_t)most - 1);
    }
}

// How far the bounds separate a snapshot's groups, measured once per load (the
// loads are synchronous): of up to kSpreadP prefills, the groups that remain
// after the K-th best cost, for requests of spread_tokens tokens, once without
// a resident prefix and once bounded as if half of it were resident somewhere.
// The mean of the two is near the groups per request that real batches leave
// (fat trees 1 to 2 of 48 groups measured, 1.0 to 1.4 here; all decodes on one
// tier under random congestion 10 to 29, 25 here; identical decodes 48, 48).
// It only chooses between forms with the same results, so updates of a loaded
// snapshot (set or smoothed congestion, committed batches) and the policy are not
// measured again.
constexpr uint32_t kSpreadP = 64, kSpreadLens = 3, kSpreadKs = 4;   // K = 1, 2, 4, 8
constexpr uint32_t kSpreadWords = kSpreadLens * kSpreadKs;
__host__ __device__ constexpr uint32_t spread_tokens(uint32_t i) { return 2048u << (3 * i); }   // 2 K, 16 K, 128 K

// One workgroup per (prefill, length), which writes its own counts for the host
// to add.  It is bound by its chain of dependent loads, 6.6 us (16.7 with the
// per-pair divisions of the other kernels, whose operands are loaded by tier).
constexpr uint32_t kSpreadWaves = 16;

template <bool TWO>
__global__ __launch_bounds__(kSpreadWaves * kWave) void spread_kernel(Snap s, const uint8_t *__restrict__ t1,
                                                                      const float *__restrict__ u1,
                                                                      const uint8_t *__restrict__ t2,
                                                                      const float *__restrict__ u2, uint32_t ngroup,
                                                                      uint32_t *__restrict__ out) {
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    __shared__ uint32_t lb[2][kBoundMaxGroups], best[kSpreadWaves * 4];
    const uint32_t lane = threadIdx.x % kWave, wv = wave_index();
    const uint32_t p = (uint32_t)((uint64_t)blockIdx.x * s.P / gridDim.x);
    const float x = (float)spread_tokens(blockIdx.y);
    // (nearly the feasibility limits: an estimate does without 64-bit divisions)
    const float per_byte = 1.0f / (float)max(s.bpt, 1u);
    // seconds per token by tier without congestion (as sec_per_token, the divisions
    // in another order), so that the loads of the loop do not depend on each other
    auto per_token = [&](uint32_t t, bool own) {
        const float n = own && s.policy < 2 ? (float)s.n_inflight[t * s.P + p] : 0.0f;
        return (float)s.bpt * (1.0f + n) / s.bw[t];
    };
    const float y0 = per_token(0, true), y1 = per_token(1, true), y2 = per_token(2, true), y3 = per_token(3, true);
    const float z0 = TWO ? per_token(0, false) : 0.0f, z1 = TWO ? per_token(1, false) : 0.0f;
    const float z2 = TWO ? per_token(2, false) : 0.0f, z3 = TWO ? per_token(3, false) : 0.0f;
    auto pick = [&](uint32_t t, float e0, float e1, float e2, float e3) {
        const float l = (t & 1u) ? e1 : e0, h = (t & 1u) ? e3 : e2;
        return (t & 2u) ? h : l;
    };
    auto rise = [&](float c) { return s.policy >= 1 ? 1.0f : __builtin_amdgcn_rcpf(1.0f - c); };
    uint32_t top[4] = {kNone, kNone, kNone, kNone};   // the thread's costs, at most four, ascending
    for (uint32_t g = wv; g < ngroup; g += kSpreadWaves) {
        const uint32_t d = g * kWave + lane;
        float2 a = make_float2(__builtin_inff(), __builtin_inff()), b = a;
        float lim = 0.0f;
        if (d < s.D) {
            const uint64_t i = (uint64_t)p * s.D + d, m = s.free_mem[d];
            const float base = load_term(s, d);
            const uint32_t tau = s.tier_map[i] & 3u;
            a = make_float2(pick(tau, y0, y1, y2, y3) * rise(s.util[i]), tier_latency(s, tau) + base);
            if (TWO) {
                const uint32_t v = t1[i] & 3u, w = t2[i] & 3u;
                b = make_float2(pick(v, y0, y1, y2, y3) * rise(u1[i]) + pick(w, z0, z1, z2, z3) * rise(u2[i]),
                                tier_latency(s, v) + tier_latency(s, w) + base);
            }
            lim = m < s.m_min ? 0.0f : fmaf((float)(m - s.m_min), per_byte, 1.0f);
        }
        uint32_t c = x < lim ? route_cost<TWO>(x, a, b) : kNone;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t lo = min(top[u], c);
            c = max(top[u], c);
            top[u] = lo;
        }
        uint32_t m[4];
        wave_min4_u32(__float_as_uint(a.x), __float_as_uint(a.y), __float_as_uint(b.x), __float_as_uint(b.y), m);
        const float2 la = make_float2(__uint_as_float(m[0]), __uint_as_float(m[1]));
        const float2 lo = make_float2(__uint_as_float(m[2]), __uint_as_float(m[3]));
        const bool f = __any(x < lim), hf = __any(0.5f * x < lim);
        if (lane == 0) {
            lb[0][g] = f ? route_cost<TWO>(x, la, lo) : kNone;
            lb[1][g] = hf ? route_cost<TWO>(0.5f * x, la, lo) : kNone;
        }
    }
    // the least of the wavefront's ascending t, taken out of the lane that has it
    auto pop = [&](uint32_t (&t)[4]) {
        const uint32_t mn = wave_min_u32_dpp(t[0]);
        if (mn != kNone && lane == (uint32_t)__builtin_ctzll(ballot(t[0] == mn))) {
            t[0] = t[1];
            t[1] = t[2];
            t[2] = t[3];
            t[3] = kNone;
        }
        return mn;
    };
    // four of each wavefront: eight of one group alone are counted as four, which
    // leaves the eighth least cost a little too high
#pragma unroll 1
    for (uint32_t u = 0; u < 4; ++u) {
        const uint32_t mn = pop(top);
        if (lane == 0) best[wv * 4 + u] = mn;
    }
    __syncthreads();
    if (wv != 0) return;
    uint32_t head[4] = {best[lane], kNone, kNone, kNone};
    const uint32_t l0 = lane < ngroup ? lb[0][lane] : kNone, l1 = lane < ngroup ? lb[1][lane] : kNone;
#pragma unroll 1
    for (uint32_t u = 0; u < 8; ++u) {
        const uint32_t kth = pop(head);
        const uint32_t n = (uint32_t)__builtin_popcountll(ballot(l0 != kNone && l0 <= kth)) +
                           (uint32_t)__builtin_popcountll(ballot(l1 != kNone && l1 <= kth));
        // (none with fewer than u + 1 feasible decodes)
        if (((u + 1) & u) == 0 && lane == 0)
            out[blockIdx.x * kSpreadWords + blockIdx.y * kSpreadKs + (uint32_t)__builtin_ctz(u + 1)] = kth != kNone ? n : kNone;
    }
}

// Holder values of the leading held blocks of every request, L neighbouring
// lanes per request, U blocks each per step with their loads issued together
// (the kernel is bound by the number of dependent loads per wavefront), and
// their count (kNoPre for an invalid request).  Steps go through the shared
// index, which stays in cache, so the blocks looked up past the run's end
// cost no memory access; the first block it does not have is looked up in
// the whole index, two lines of it from memory, and only where that block
// has one holder do the following steps go there.
template <uint32_t L, uint32_t U>
__global__ __launch_bounds__(kBlock) void match_kernel(Snap s, Table t, Shared sh, Reqs rq,
                                                       uint32_t *__restrict__ hv, uint32_t *__restrict__ mm,
                                                       uint32_t *__restrict__ err) {
    const uint32_t lane = threadIdx.x % kWave, sub = lane % L, seg0 = lane - sub;
    const uint64_t r = (uint64_t)blockIdx.x * (kBlock / L) + threadIdx.x / L;
    const bool in = r < rq.n_req;
    uint32_t p, len, n = 0;
    uint64_t a = 0;
    const bool ok = in && request_ok(rq, s, (uint32_t)r, p, len, a, n);
    if (!ok) n = 0;
    uint32_t m = n;
    bool act = n > 0;
    // blocks from k on through an index, up to the first it does not have
    // (past the run's end: a miss, so m is at most n); after kAlone blocks the
    // whole wavefront takes one request after another, as many blocks per step
    // in all (a wavefront with one run of 4,096 held blocks takes 30 steps
    // more, and not 240)
    constexpr uint32_t kAlone = 256;
    auto steps = [&](auto lookup, uint32_t k) {
        for (uint32_t done = 0; __any(act) && done < kAlone; done += L * U, k += L * U) {
            uint64_t h[U];
            uint32_t v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t kk = k + u * L + sub;
                h[u] = act && kk < n ? rq.hashes[a + kk] : 0ull;   // hash 0 is held nowhere
            }
            lookup(h, v);
            uint32_t first = L * U;
#pragma unroll
            for (int u = (int)U - 1; u >= 0; --u) {
                const uint32_t miss = (uint32_t)(ballot(v[u] == kNoHolder) >> seg0) & (uint32_t)((1ull << L) - 1);
                if (miss) first = (uint32_t)u * L + (uint32_t)__builtin_ctz(miss);
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if (act && u * L + sub < first) hv[a + k + u * L + sub] = v[u];
            if (act && first < L * U) {
                m = k + first;
                act = false;
            }
        }
        for (lmask left = ballot(act && sub == 0); left; left &= left - 1) {
            const uint32_t l = (uint32_t)__builtin_ctzll(left);
            const uint32_t nl = (uint32_t)__builtin_amdgcn_readlane((int)n, (int)l);
            const uint64_t al = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(a >> 32), (int)l) << 32) |
                                (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)a, (int)l);
            uint32_t kl = (uint32_t)__builtin_amdgcn_readlane((int)k, (int)l), first = kWave * U;
            for (;; kl += kWave * U) {
                uint64_t h[U];
                uint32_t v[U];
#pragma unroll
                for (uint32_t u = 0; u < U; ++u) {
                    const uint32_t kk = kl + u * kWave + lane;
                    h[u] = kk < nl ? rq.hashes[al + kk] : 0ull;
                }
                lookup(h, v);
                first = kWave * U;
#pragma unroll
                for (int u = (int)U - 1; u >= 0; --u) {
                    const lmask miss = ballot(v[u] == kNoHolder);
                    if (miss) first = (uint32_t)u * kWave + (uint32_t)__builtin_ctzll(miss);
                }
#pragma unroll
                for (uint32_t u = 0; u < U; ++u)
                    if (u * kWave + lane < first) hv[al + kl + u * kWave + lane] = v[u];
                if (first < kWave * U) break;   // (at the run's end at the latest)
            }
            if (seg0 == l) {
                m = kl + first;
                act = false;
            }
        }
    };
    uint32_t k = 0;
    if (sh.b) {
        steps(
            [&](const uint64_t (&h)[U], uint32_t (&v)[U]) {
                uint32_t i[U];
                u32x4 x[U];
#pragma unroll
                for (uint32_t u = 0; u < U; ++u) {
                    i[u] = shared_slot(sh, h[u]);
                    x[u] = u32x4{0, 0, 0, 0};
                    if (h[u]) x[u] = sh.b[i[u]];
                }
#pragma unroll
                for (uint32_t u = 0; u < U; ++u) v[u] = shared_find(sh, h[u], i[u], x[u]);
            },
            0);
        uint32_t v = kNoHolder;
        if (sub == 0 && m < n) v = holder_lane_lean(t, rq.hashes[a + m]);
        if (v != kNoHolder) hv[a + m] = v;
        act = ((ballot(v != kNoHolder) >> seg0) & 1ull) != 0;
        if (act) {
            k = m + 1;
            m = n;
        }
    }
    steps(
        [&](const uint64_t (&h)[U], uint32_t (&v)[U]) {
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) v[u] = holder_lane(t, h[u]);
        },
        k);
    if (in && sub == 0) mm[r] = ok ? m : kNoPre;
    if (ballot(in && !ok) && threadIdx.x % kWave == 0) atomicOr(err, kErrRequest);
}

// Leading words of this wavefront's `word`s (lane k: block k's, zero past the
// run) that hold each lane's bit, 0 .. 64 (few: fewer than 16 words are not
// zero).  An inclusive AND over the lanes leaves the decodes that hold every
// block up to k in lane k; a lane's count is found by a binary search over
// the words in LDS, of which it reads the half with its bit.  20 vector
// instructions for short runs, 33 for long ones, and no scalar ones (a loop
// over the blocks with read-lanes took 3 vector and 8 scalar instructions a
// block, and the scalar unit bound the kernel).
// The array holds 32-bit words, low and high halves in turn, as they are read:
// stored as 64-bit ones, the compiler may take stores and reads as unrelated.
__device__ inline uint32_t leading_words(uint32_t *wds, uint64_t word, uint32_t lane, bool few) {
    uint32_t lo = (uint32_t)word, hi = (uint32_t)(word >> 32);
    lo &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)lo, 0x111, 0xF, 0xF, false);   // row_shr 1
    hi &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)hi, 0x111, 0xF, 0xF, false);
    lo &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)lo, 0x112, 0xF, 0xF, false);
    hi &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)hi, 0x112, 0xF, 0xF, false);
    lo &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)lo, 0x114, 0xF, 0xF, false);
    hi &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)hi, 0x114, 0xF, 0xF, false);
    lo &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)lo, 0x118, 0xF, 0xF, false);
    hi &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)hi, 0x118, 0xF, 0xF, false);
    if (!few) {
        lo &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)lo, 0x142, 0xA, 0xF, false);   // row_bcast 15
        hi &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)hi, 0x142, 0xA, 0xF, false);
        lo &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)lo, 0x143, 0xC, 0xF, false);   // row_bcast 31
        hi &= (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)hi, 0x143, 0xC, 0xF, false);
    }
    lane_phase();
    wds[2 * lane] = lo;
    wds[2 * lane + 1] = hi;
    lane_phase();
    const uint32_t *half = wds + (lane >> 5);
    const uint32_t sh = lane & 31u;
    uint32_t j = 0;
    if (!few) {
        j += ((half[2 * (j + 31)] >> sh) & 1u) << 5;
        j += ((half[2 * (j + 15)] >> sh) & 1u) << 4;
    }
    j += ((half[2 * (j + 7)] >> sh) & 1u) << 3;
    j += ((half[2 * (j + 3)] >> sh) & 1u) << 2;
    j += ((half[2 * (j + 1)] >> sh) & 1u) << 1;
    j += (half[2 * j] >> sh) & 1u;
    if (!few) j += (half[2 * j] >> sh) & 1u;   // 63 found so far: the last word
    return j;
}

// Each wavefront takes `per` (1, 2 or a multiple of 4, at most 64 / K)
// consecutive requests, four at a time with their loads issued together; the
// results are gathered one per lane and stored at the end.
template <int K, bool TWO>
__global__ __launch_bounds__(kBlock) void bounded_kernel(Snap s, Table t, Reqs rq, Bounds bd,
                                                         const uint32_t *__restrict__ hv,
                                                         const uint32_t *__restrict__ mm, uint32_t per, uint32_t k_out,
                                                         int32_t *__restrict__ out_idx, float *__restrict__ out_score) {
    constexpr int Q = 4;
    __shared__ __align__(8) uint32_t lds[kWavesPerBlock][Q][2 * kWave];
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t wv = wave_index();
    const uint64_t first = ((uint64_t)blockIdx.x * kWavesPerBlock + wv) * per;
    if (first >= rq.n_req) return;
    const uint32_t r0 = (uint32_t)first;
    const uint32_t cnt = rq.n_req - r0 < per ? rq.n_req - r0 : per;
    const uint32_t bt = s.block_tokens, ng = bd.ngroup;
    const float xgl = lane < ng ? bd.xg[lane] : -1.0f;
    const uint32_t lg = lane < ng ? lane : 0u;
    uint32_t res_b = 0xFFFFFFFFu, res_d = 0xFFFFFFFFu;   // K keys per request, request i's from lane i * K
    for (uint32_t i0 = 0; i0 < cnt; i0 += Q) {
        uint32_t p[Q], len[Q], m[Q], mq[Q];
        uint64_t a[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint32_t r = r0 + (i0 + q < cnt ? i0 + q : i0);
            m[q] = as_const(mm)[r];
            p[q] = as_const(rq.prefill)[r];
            len[q] = as_const(rq.len)[r];
            a[q] = as_const(rq.off)[r];
        }
        // bounds of the groups (lane g: group g), and the leading holder
        // values (lane k: block k); an invalid request is scored as one
        // without blocks and its result dropped
        float2 b1[Q], b2[Q];
        uint32_t v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            mq[q] = m[q] == kNoPre ? 0u : m[q];
            if (m[q] == kNoPre) p[q] = 0;
            b1[q] = (bd.lo + (uint64_t)p[q] * ng)[lg];
            if (TWO) b2[q] = (bd.lo2 + (uint64_t)p[q] * ng)[lg];
            v[q] = kNoHolder;
            if (lane < mq[q]) v[q] = (hv + a[q])[lane];
        }
        uint32_t lb[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const float xlo = (float)(len[q] - bt * mq[q]);
            uint32_t c = __float_as_uint(fmaf(xlo, b1[q].x, b1[q].y));
            if (TWO) c = min(c, __float_as_uint(fmaf(xlo, b2[q].x, b2[q].y)));
            // (requests of 2^24 tokens or more: the limits are capped there)
            lb[q] = lane < ng && (xlo <= xgl || len[q] >= kExactTok) ? c : 0xFFFFFFFFu;
        }
        uint32_t least[Q];
        wave_min4_u32(lb[0], lb[1], lb[2], lb[3], least);
        // the group of least bound of each request: its rows, words and limits
        auto words = [&](uint32_t g, uint32_t v_) -> uint64_t {
            uint64_t wd = 0;
            if (v_ < kHeldOne) wd = t.bits[(uint64_t)v_ * t.bpitch + g];
            else if (v_ != kNoHolder && (v_ & ~kHeldOne) / kWave == g) wd = 1ull << ((v_ & ~kHeldOne) % kWave);
            return wd;
        };
        uint32_t home[Q];
        float2 row[Q], row2[Q];
        float xm[Q];
        uint64_t word[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            // (no group can take it: lane 0, where nothing is feasible)
            home[q] = (uint32_t)__builtin_ctzll(ballot(lb[q] == least[q]));
            const uint64_t o = (uint64_t)p[q] * s.slp + home[q] * kWave;   // (past D: padding or the next row)
            row[q] = (s.sl + o)[lane];
            if (TWO) row2[q] = (s.sr + o)[lane];
            xm[q] = (bd.xm + home[q] * kWave)[lane];
            word[q] = words(home[q], v[q]);
        }
        // the lane's cost bits of request q on its decode of group g
        auto cost = [&](int q, uint32_t g, float2 x1, float2 x2, float lim, uint64_t wd) -> uint32_t {
            uint32_t j = leading_words(lds[wv][q], wd, lane, mq[q] < 16);
            for (uint32_t k0 = kWave; k0 < mq[q] && __any(j == k0); k0 += 2 * kWave) {   // runs of more than 64 held blocks
                const uint32_t v0 = k0 + lane < mq[q] ? (hv + a[q] + k0)[lane] : kNoHolder;
                const uint32_t v1 = k0 + kWave + lane < mq[q] ? (hv + a[q] + k0 + kWave)[lane] : kNoHolder;
                const uint64_t w0 = words(g, v0), w1 = words(g, v1);
                uint32_t more = leading_words(lds[wv][q], w0, lane, mq[q] - k0 < 16);
                if (mq[q] - k0 > (uint32_t)kWave) {
                    const uint32_t next = leading_words(lds[wv][q], w1, lane, mq[q] - k0 - kWave < 16);
                    more += more == (uint32_t)kWave ? next : 0u;
                }
                j += j == k0 ? more : 0u;
            }
            const uint32_t x = len[q] - bt * j;
            const float xf = (float)x;
            bool feas = xf <= lim;
            if (len[q] >= kExactTok) {
                const uint32_t d = g * kWave + lane;
                feas = d < s.D && (uint64_t)x < s.dxlim[d < s.D ? d : 0u];
            }
            const uint32_t c = route_cost<TWO>(xf, x1, x2);
            return feas ? c : 0xFFFFFFFFu;
        };
        uint32_t cb[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) cb[q] = cost(q, home[q], row[q], row2[q], xm[q], word[q]);
        uint32_t best[Q];
        wave_min4_u32(cb[0], cb[1], cb[2], cb[3], best);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (i0 + q >= cnt) continue;
            // keys kept: lanes 0 .. K-1 of kb / kd, ascending (cost bits, decode)
            uint32_t kb = 0xFFFFFFFFu, kd = 0xFFFFFFFFu;
            uint32_t thr;   // k-th best cost bits
            if (K == 1) {
                thr = best[q];
                kb = best[q];
                if (best[q] != 0xFFFFFFFFu) kd = home[q] * kWave + (uint32_t)__builtin_ctzll(ballot(cb[q] == best[q]));
            }
            // merge the column of group g into the kept keys
            auto merge = [&](uint32_t g, uint32_t c) {
                uint32_t ob = kb, od = kd;   // the old keys, consumed as they are placed
                uint32_t nb = 0xFFFFFFFFu, nd = 0xFFFFFFFFu;
                const uint32_t dl = g * kWave + lane;
#pragma unroll
                for (int u = 0; u < K; ++u) {
                    const uint32_t mn = wave_min_u32_dpp(min(c, ob));
                    if (mn == 0xFFFFFFFFu) break;
                    const uint32_t dm = wave_min_u32_dpp(min(c == mn ? dl : 0xFFFFFFFFu, ob == mn ? od : 0xFFFFFFFFu));
                    if (c == mn && dl == dm) c = 0xFFFFFFFFu;
                    if (ob == mn && od == dm) ob = 0xFFFFFFFFu;
                    nb = write_lane(mn, (uint32_t)u, nb);
                    nd = write_lane(dm, (uint32_t)u, nd);
                }
                kb = nb;
                kd = nd;
            };
            if (K > 1) {
                if (best[q] != 0xFFFFFFFFu) merge(home[q], cb[q]);
                thr = (uint32_t)__builtin_amdgcn_readlane((int)kb, (int)k_out - 1);
            }
            lmask left = ballot(lb[q] <= thr && lb[q] != 0xFFFFFFFFu) & ~(1ull << home[q]);
            while (left) {
                const uint32_t g = (uint32_t)__builtin_ctzll(left);
                const uint64_t o = (uint64_t)p[q] * s.slp + g * kWave;
                const float2 x1 = (s.sl + o)[lane];
                const float2 x2 = TWO ? (s.sr + o)[lane] : x1;
                const uint32_t c = cost(q, g, x1, x2, (bd.xm + g * kWave)[lane], words(g, v[q]));
                if (K == 1) {
                    const uint32_t mn = wave_min_u32_dpp(c);
                    if (mn <= thr && mn != 0xFFFFFFFFu) {
                        const uint32_t dm = g * kWave + (uint32_t)__builtin_ctzll(ballot(c == mn));
                        if (mn < thr || dm < kd) kd = dm;
                        thr = mn;
                        kb = mn;
                    }
                } else if (ballot(c <= thr && c != 0xFFFFFFFFu)) {
                    merge(g, c);
                    thr = (uint32_t)__builtin_amdgcn_readlane((int)kb, (int)k_out - 1);
                }
                left &= left - 1;
                left &= ballot(lb[q] <= thr);
            }
            const uint32_t slot = (i0 + q) * K;
            if (m[q] == kNoPre) {   // marks an invalid request: no cost has these bits with a decode
                res_b = write_lane(0xFFFFFFFEu, slot, res_b);
            } else if (K == 1) {
                res_b = write_lane(kb, slot, res_b);
                res_d = write_lane(kd, slot, res_d);
            } else {
#pragma unroll
                for (int u = 0; u < K; ++u) {
                    res_b = write_lane((uint32_t)__builtin_amdgcn_readlane((int)kb, u), slot + u, res_b);
                    res_d = write_lane((uint32_t)__builtin_amdgcn_readlane((int)kd, u), slot + u, res_d);
                }
            }
        }
    }
    // lane i * K + u: key u of request i
    const uint32_t i = lane / K, u = lane % K;
    const uint32_t headb = (uint32_t)__shfl((int)res_b, (int)(i * K), kWave);
    if (i < cnt && u < k_out) {
        const bool bad = headb == 0xFFFFFFFEu, none = res_b == 0xFFFFFFFFu;
        const uint64_t o = (uint64_t)(r0 + i) * k_out + u;
        out_idx[o] = bad || none ? -1 : (int32_t)res_d;
        out_score[o] = bad ? __builtin_nanf("") : none ? __builtin_inff() : __uint_as_float(res_b);
    }
}

// ---------------------------------------------------------------- ranking sweep
//
// Re-ranking of a batch under congestion scenarios (Sec. V-D).  Prefix
// lengths do not depend on congestion: every request's non-cached tokens on
// every decode come from its scoring record (leader row and cap, as in
// score_kernel) once, and only seconds per token change per scenario.
// Under scenario s the pair costs x * spt_s(p, d) + (L + load term), with
// spt_s from the scenario's congestion by the same expression as the
// snapshot's derived rows, so a scenario equal to the snapshot reproduces
// the selection bit for bit.

// Seconds per non-cached token of every (scenario, p, d).
__global__ __launch_bounds__(256) void derive_scen_kernel(Snap s, const float *__restrict__ util_scen, uint64_t n,
                                                          float *__restrict__ spt) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t pd = i % ((uint64_t)s.P * s.D);
    const uint32_t p = (uint32_t)(pd / s.D);
    spt[i] = sec_per_token(s, s.tier_map[pd] & 3u, p, util_scen[i]);
}

constexpr uint32_t kSweepThreads = 256;   // requests per workgroup, one per thread, in batch order
constexpr uint32_t kSweepScen = 32;       // scenarios per workgroup
constexpr uint32_t kSweepMaxTab = 8192;   // largest P * Dp kept in LDS (two fp32 tables; three when held)
constexpr uint32_t kSweepHold = 3;        // scenario-table entries a thread holds while the previous is scored

// Ascending top-K list of fp32 cost bits (unsigned order) and decodes:
// insert (key, d) by min / median-of-three on the values and selects on the
// indices; decodes come in ascending order and only a strictly smaller key
// moves ahead, so equal costs keep the lower index first.
template <int K>
__device__ inline void topk_ins32(uint32_t (&t)[K], uint32_t (&ix)[K], uint32_t key, uint32_t d) {
    bool c[K];
#pragma unroll
    for (int q = 0; q < K; ++q) c[q] = key < t[q];
#pragma unroll
    for (int q = K - 1; q >= 1; --q) {
        ix[q] = c[q - 1] ? ix[q - 1] : (c[q] ? d : ix[q]);
        // the median of t[q-1], t[q] and key, in the form the compiler
        // turns into one median-of-three instruction
        t[q] = max(min(t[q - 1], t[q]), min(max(t[q - 1], t[q]), key));
    }
    ix[0] = c[0] ? d : ix[0];
    t[0] = min(t[0], key);
}

// Decodes db .. db+63 holding a hash with holder value v, as a bit mask
// (db a multiple of 64, or 0).
__device__ inline uint64_t held_mask(const Table &t, uint32_t v, uint32_t db) {
    if (v == kNoHolder) return 0;
    if (v & kHeldOne) {
        const uint32_t o = (v & ~kHeldOne) - db;
        return o < (uint32_t)kWave ? 1ull << o : 0ull;
    }
    return t.bits[(uint64_t)v * t.bpitch + db / kWave];
}

// Non-cached tokens x of the lane's request on decodes db .. db+NX-1, as
// fp32, -inf where infeasible.  From the leader row (min with the cap), or
// for a request marked to match on its own, a first-miss scan of its run in
// integers (x then rounded to fp32, as the scoring kernel does).
template <int NX>
__device__ inline void sweep_x(const Snap &s, const Table &t, const Reqs &rq, const Hot &rec, uint32_t r,
                               const float *lead_lam, uint32_t db, float (&xf)[NX]) {
    if ((int32_t)rec.lams >= 0) {
        const float lenf = __uint_as_float(rec.len);
        const float *row = lead_lam + rec.lrow / sizeof(float);
#pragma unroll
        for (int u = 0; u < NX; ++u) {
            const uint32_t d = db + u;
            float x = -__builtin_inff();
            if (d < s.D) {
                const uint64_t xlim = s.dxlim[d];
                const float xm = xlim == 0 ? -1.0f : (float)(xlim - 1 < kExactTok ? xlim - 1 : (uint64_t)kExactTok);
                const float lam = __uint_as_float(min(__float_as_uint(row[d]), rec.lams));
                const float xx = lenf - lam;
                x = xx <= xm ? xx : -__builtin_inff();
            }
            xf[u] = x;
        }
        return;
    }
    uint32_t p, len, n;
    uint64_t a;
    request_ok(rq, s, r, p, len, a, n);   // validated by the selection
    uint32_t jx[NX];
#pragma unroll
    for (int u = 0; u < NX; ++u) jx[u] = n;
    uint64_t alive = ~0ull;
    for (uint32_t b = 0; b < n && alive; ++b) {
        const uint64_t dead = alive & ~held_mask(t, holder_lane(t, rq.hashes[a + b]), db);
#pragma unroll
        for (int u = 0; u < NX; ++u) jx[u] = (dead >> u) & 1ull ? b : jx[u];
        alive &= ~dead;
    }
#pragma unroll
    for (int u = 0; u < NX; ++u) {
        const uint32_t d = db + u;
        float x = -__builtin_inff();
        if (d < s.D) {
            const uint32_t xi = len - s.block_tokens * jx[u];
            x = (uint64_t)xi < s.dxlim[d] ? (float)xi : -__builtin_inff();
        }
        xf[u] = x;
    }
}

// One thread per request (batch order), kSweepScen scenarios per
// workgroup.  LDS: the (L + load term) constants of every (p, d) and two
// buffers of one scenario's seconds per token, rows of Dp = D | 1 (an odd
// pitch, so lanes of different prefills read different banks).  While a
// scenario is scored from one buffer, each thread holds its share of the
// next scenario's table (loaded before the scoring, at most kSweepHold
// entries) and stores it into the other buffer afterwards, so one barrier
// per scenario suffices and the loads' latency is hidden behind the
// scoring; larger tables are copied before each scenario instead.  NX decodes'
// tokens are held in registers; a pool of more decodes is taken NX at a
// time and its tokens recomputed per scenario.  FULL: exactly NX decodes,
// every decode index a compile-time constant (no bounds test per pair).
// Writes the top-k of every scenario and counts, per scenario, the requests
// whose selected tier / decode differs from the loaded snapshot's selection.
template <int K, int NX, bool LDS, bool FULL>
__global__ __launch_bounds__(kSweepThreads, FULL ? (K == 1 ? 6 : 5) : 1) void sweep_kernel(Snap s, Table t, Reqs rq, const Hot *__restrict__ hotr,
                                                             const float *__restrict__ lead_lam,
                                                             const float *__restrict__ spt_scen, uint32_t n_scen,
                                                             const int32_t *__restrict__ base_idx,
                                                             const float *__restrict__ base_score, uint32_t k_out,
                                                             int32_t *__restrict__ out_idx,
                                                             float *__restrict__ out_score,
                                                             unsigned long long *__restrict__ flips) {
    extern __shared__ float tab[];   // LDS: [P][Dp] constants, then 2 x [P][Dp] seconds per token
    const uint32_t P = s.P, D = FULL ? (uint32_t)NX : s.D, Dp = D | 1u;
    const uint32_t r = blockIdx.x * kSweepThreads + threadIdx.x;
    const uint32_t s0 = blockIdx.y * kSweepScen;
    const uint32_t s1 = min(s0 + kSweepScen, n_scen);
    const bool act = r < rq.n_req;
    const bool valid = act && !__builtin_isnan(base_score[r]);
    Hot rec = Hot{0, 0, 0, 0};
    uint32_t p = 0;
    if (valid) {
        rec = hotr[r];
        p = rec.row / (s.slp * (uint32_t)sizeof(float2));
    }
    float *tc = tab, *tsb = tab + (uint64_t)P * Dp;
    // a scenario's seconds per token into LDS buffer b (all of them, by
    // this workgroup's threads)
    auto table_copy = [&](uint32_t sc, uint32_t b) {
        const float *sp = spt_scen + (uint64_t)sc * P * D;
        float *ts = tsb + (uint64_t)b * P * Dp;
        for (uint32_t i = threadIdx.x; i < P * D; i += kSweepThreads) {
            const uint32_t pp = i / D;
            ts[pp * Dp + (i - pp * D)] = sp[i];
        }
    };
    const bool held = P * D <= kSweepThreads * kSweepHold;
    if (LDS) {
        for (uint32_t i = threadIdx.x; i < P * D; i += kSweepThreads) {
            const uint32_t pp = i / D, d = i - pp * D;
            tc[pp * Dp + d] = s.sl[(uint64_t)pp * s.slp + d].y;
        }
        if (held && s0 < s1) table_copy(s0, 0);
    }
    const bool one = FULL || D <= (uint32_t)NX;
    float xf[NX];
    if (valid && one) sweep_x<NX>(s, t, rq, rec, r, lead_lam, 0, xf);
    const int32_t bsel = valid ? base_idx[r] : -1;
    const int btier = bsel < 0 ? -1 : (int)(s.tier_map[(uint64_t)p * D + (uint32_t)bsel] & 3u);
    const uint32_t lrow = p * Dp;
    for (uint32_t sc = s0; sc < s1; ++sc) {
        const float *sp = spt_scen + (uint64_t)sc * P * D;
        const uint32_t buf = held ? (sc - s0) & 1u : 0u;
        const float *ts = tsb + (uint64_t)buf * P * Dp;
        float nx[kSweepHold];   // this thread's share of the next scenario's table
        if (LDS) {
            if (held) {
                __syncthreads();   // this scenario's buffer is written and the other one no longer read
                if (sc + 1 < s1) {
                    const float *spn = sp + (uint64_t)P * D;
#pragma unroll
                    for (uint32_t h = 0; h < kSweepHold; ++h) {
                        const uint32_t i = threadIdx.x + h * kSweepThreads;
                        nx[h] = i < P * D ? spn[i] : 0.0f;
                    }
                }
            } else {
                __syncthreads();   // the previous scenario's table is no longer read
                table_copy(sc, 0);
                __syncthreads();
            }
        }
        uint32_t tk[K], ti[K];
#pragma unroll
        for (int q = 0; q < K; ++q) {
            tk[q] = 0xFFFFFFFFu;
            ti[q] = 0xFFFFFFFFu;
        }
        if (valid) {
            if (FULL) {
#pragma unroll
                for (int u = 0; u < NX; ++u) {
                    const float spt = LDS ? ts[lrow + u] : sp[(uint64_t)p * D + u];
                    const float cst = LDS ? tc[lrow + u] : s.sl[(uint64_t)p * s.slp + u].y;
                    topk_ins32<K>(tk, ti, __float_as_uint(fmaf(xf[u], spt, cst)), (uint32_t)u);
                }
            } else {
                for (uint32_t db = 0; db < D; db += NX) {
                    if (!one) sweep_x<NX>(s, t, rq, rec, r, lead_lam, db, xf);
#pragma unroll
                    for (int u = 0; u < NX; ++u) {
                        const uint32_t d = db + u;
                        if (d < D) {
                            const float spt = LDS ? ts[lrow + d] : sp[(uint64_t)p * D + d];
                            const float cst = LDS ? tc[lrow + d] : s.sl[(uint64_t)p * s.slp + d].y;
                            topk_ins32<K>(tk, ti, __float_as_uint(fmaf(xf[u], spt, cst)), d);
                        }
                    }
                }
            }
        }
        if (LDS && held && sc + 1 < s1) {
            float *tn = tsb + (uint64_t)(buf ^ 1u) * P * Dp;
#pragma unroll
            for (uint32_t h = 0; h < kSweepHold; ++h) {
                const uint32_t i = threadIdx.x + h * kSweepThreads;
                if (i < P * D) {
                    const uint32_t pp = i / D;
                    tn[pp * Dp + (i - pp * D)] = nx[h];
                }
            }
        }
        uint32_t tier_flip = 0, idx_flip = 0;
        if (act) {
            const uint64_t o = ((uint64_t)sc * rq.n_req + r) * k_out;
#pragma unroll
            for (int q = 0; q < K; ++q) {
                if ((uint32_t)q < k_out) {
                    // a key with its sign bit set is an infeasible pair (cost -inf)
                    const bool none = !valid || tk[q] >= 0x80000000u;
                    out_idx[o + q] = none ? -1 : (int32_t)ti[q];
                    out_score[o + q] = !valid ? __builtin_nanf("") : none ? __builtin_inff() : __uint_as_float(tk[q]);
                }
            }
            if (valid) {
                const int32_t sel = tk[0] >= 0x80000000u ? -1 : (int32_t)ti[0];
                const int ts_ = sel < 0 ? -1 : (int)(s.tier_map[(uint64_t)p * D + (uint32_t)sel] & 3u);
                tier_flip = ts_ != btier;
                idx_flip = sel != bsel;
            }
        }
        if (flips) {
            const uint32_t fa = wave_sum_u32(tier_flip), fb = wave_sum_u32(idx_flip);
            if ((threadIdx.x % kWave) == 0) {
                if (fa) atomicAdd(flips + 2 * sc, (unsigned long long)fa);
                if (fb) atomicAdd(flips + 2 * sc + 1, (unsigned long long)fb);
            }
        }
    }
}

// Proposition 2 (Sec. V-D) per scenario: pairs of decodes on different
// tiers from one prefill instance, their bandwidths X = B'(1 - c) with
// B' = B_tau / (1 + n_inflight[tau][p]) under the snapshot's congestion and
// under the scenario's, counted into out[3 s + 0..2]: pairs the
// proposition's sufficient condition covers (the larger of the two
// congestion errors below |X - X'| / (B'_tau + B'_tau')), inverted pairs
// among them, all inverted pairs (the snapshot's strict order not kept).
// fp64, every operation in a fixed order, so the counts are exact.  One
// thread per (p, d), pairs with the decodes after d.
struct Bw64 {
    double b[4];
};

__global__ __launch_bounds__(256) void tier_inv_kernel(Snap s, Bw64 bw, const float *__restrict__ util_scen,
                                                       unsigned long long *__restrict__ out) {
    const uint32_t sc = blockIdx.y;
    const uint64_t pd = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t npd = (uint64_t)s.P * s.D;
    uint32_t covered = 0, inv_cov = 0, inverted = 0;
    if (pd < npd) {
        const uint32_t p = (uint32_t)(pd / s.D), d = (uint32_t)(pd - (uint64_t)p * s.D);
        const float *u = util_scen + (uint64_t)sc * npd;
        // B' of each tier for this prefill (the same division for every pair)
        double bt[4];
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) bt[t] = bw.b[t] / (1.0 + (double)s.n_inflight[t * s.P + p]);
        const uint32_t ta = s.tier_map[pd] & 3u;
        const double ba = ta == 0 ? bt[0] : ta == 1 ? bt[1] : ta == 2 ? bt[2] : bt[3];
        const double ca = (double)s.util[pd], ha = (double)u[pd];
        const double xa = ba * (1.0 - ca), ya = ba * (1.0 - ha);
        for (uint32_t e = d + 1; e < s.D; ++e) {
            const uint64_t q = (uint64_t)p * s.D + e;
            const uint32_t tb = s.tier_map[q] & 3u;
            if (tb == ta) continue;
            const double bb = tb == 0 ? bt[0] : tb == 1 ? bt[1] : tb == 2 ? bt[2] : bt[3];
            const double cb = (double)s.util[q], hb = (double)u[q];
            const double xb = bb * (1.0 - cb), yb = bb * (1.0 - hb);
            if (xa == xb) continue;
            const bool inv = xa > xb ? !(ya > yb) : !(ya < yb);
            const double eps = fmax(fabs(ha - ca), fabs(hb - cb));
            const bool cov = eps < fabs(xa - xb) / (ba + bb);
            covered += cov;
            inv_cov += cov && inv;
            inverted += inv;
        }
    }
    covered = wave_sum_u32(covered);
    inv_cov = wave_sum_u32(inv_cov);
    inverted = wave_sum_u32(inverted);
    if ((threadIdx.x % kWave) == 0) {
        if (covered) atomicAdd(out + 3 * (uint64_t)sc, (unsigned long long)covered);
        if (inv_cov) atomicAdd(out + 3 * (uint64_t)sc + 1, (unsigned long long)inv_cov);
        if (inverted) atomicAdd(out + 3 * (uint64_t)sc + 2, (unsigned long long)inverted);
    }
}

// ------------------------------------------------------------------ table build

// ---- holder index build (once per cache load)
//
// The (hash, decode) pairs of all resident sets are partitioned by the top
// bits of the mixed hash (rocPRIM radix sort over those bits alone: one or two
// passes), so that the hashes of a block of buckets lie together, and the rest
// happens in LDS, one workgroup per part or block, with coalesced reads and
// writes of memory:
//   pair_kernel   -- mixed hash and decode of every resident hash;
//   parts_kernel  -- where each part starts;
//   dedupe_kernel -- a part's distinct hashes, each with one holder and whether
//                    it has more, and their counts (which size the set);
//   build_kernel  -- a block's cuckoo set, its values, the bitmap rows and the
//                    shared index.
// A whole load of 50.3 M pairs of 768 decodes takes 3.3 ms (build 1.24, dedupe
// 0.77, the sort 0.55, pairs 0.17, parts 0.12 and the allocations that are
// left), against 17.0 ms with a sort over all 64 bits, one thread per distinct
// hash walking its run of up to 768 holders, compare-and-swaps on the set in
// memory, and all buffers allocated anew.

// The largest d with off[d] <= x.
__device__ inline uint32_t owner_of(const uint64_t *__restrict__ off, uint32_t D, uint64_t x) {
    uint32_t lo = 0, hi = D;
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (off[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The pairs' sort keys: mixed values with their top `bits` bits, the part,
// rotated to the low end (the sort goes over the low bits).
__device__ inline uint64_t part_key(uint64_t x, uint32_t bits) { return (x << bits) | (x >> 1 >> (63 - bits)); }
__device__ inline uint64_t part_value(uint64_t y, uint32_t bits) { return (y >> bits) | (y << 1 << (63 - bits)); }

// Key and decode of every resident hash (binary search of the offsets, once
// per 512 hashes where those are one decode's); sets *flag when a hash is the
// reserved 0.
constexpr uint32_t kPairPer = 8;
__global__ __launch_bounds__(kBlock) void pair_kernel(const uint64_t *__restrict__ off, uint32_t D, uint64_t first,
                                                      uint64_t n, const uint64_t *hashes, uint32_t bits,
                                                      uint64_t *key, uint32_t *__restrict__ dec,
                                                      uint32_t *__restrict__ flag) {
    const uint32_t lane = threadIdx.x % kWave;
    const uint64_t i0 = ((uint64_t)blockIdx.x * kWavesPerBlock + wave_index()) * (kWave * kPairPer);
    if (i0 >= n) return;
    const uint64_t last = n - i0 < kWave * kPairPer ? n - 1 : i0 + kWave * kPairPer - 1;
    const uint32_t d0 = owner_of(off, D, first + i0), d1 = owner_of(off, D, first + last);
    bool zero = false;
#pragma unroll
    for (uint32_t u = 0; u < kPairPer; ++u) {
        const uint64_t i = i0 + u * kWave + lane;
        if (i < n) {
            const uint64_t h = hashes[i];
            zero |= h == 0;
            key[i] = part_key(mix_hash(h), bits);   // (may be the same array)
            dec[i] = d0 == d1 ? d0 : owner_of(off, D, first + i);
        }
    }
    if (__any(zero) && lane == 0) atomicOr(flag, 1u);
}

// start[q], q = 0 .. 2^bits: the first pair of part q or a later one.
__global__ __launch_bounds__(256) void parts_kernel(const uint64_t *__restrict__ key, uint64_t n, uint32_t bits,
                                                    uint32_t *__restrict__ start) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    auto part = [&](uint64_t x) { return (uint32_t)key[x] & ((1u << bits) - 1u); };
    const uint32_t lo = i == 0 ? 0u : part(i - 1) + 1u, hi = i == n ? 1u << bits : part(i);
    for (uint32_t q = lo; q <= hi; ++q) start[q] = (uint32_t)i;
}

constexpr uint32_t kBlockSlots = 2u << kBlockLog2;   // slots of a block of the set
// Most occupancy of a blocked set of several blocks.  Each block holds a random
// share of the keys, a standard deviation of 0.014 of its slots at 0.80, and
// has to stay below the two-choice threshold by itself: at 0.85 some block of
// 2^11 exceeds it in sets of 128 blocks and more, at 0.83 in sets of some
// 10,000; at 0.80 the threshold is seven standard deviations away.
constexpr double kBlockedMost = 0.80;
constexpr uint32_t kManyHolders = 0x80000000u;   // with the decode of one of them
constexpr uint32_t kNobody = 0xFFFFFFFFu;
constexpr uint32_t kShortProbe = 64;

// One workgroup per part: its distinct hashes to (okey, ohold) from the part's
// start on, count[part] of them; sums of the counts, and of the hashes of
// several holders, in cnt.  S slots hold the part's hashes at the load factor
// of the set or less on average; *flag gets 2 where they do not.
template <uint32_t S>
__global__ __launch_bounds__(1024) void dedupe_kernel(const uint64_t *__restrict__ key,
                                                      const uint32_t *__restrict__ dec,
                                                      const uint32_t *__restrict__ start, uint32_t bits,
                                                      uint64_t *__restrict__ okey,
                                                      uint32_t *__restrict__ ohold, uint32_t *__restrict__ count,
                                                      unsigned long long *__restrict__ cnt,
                                                      uint32_t *__restrict__ flag) {
    __shared__ unsigned long long lk[S];
    __shared__ uint32_t lh[S];
    __shared__ uint32_t n_out, n_many, full;
    const uint32_t a = start[blockIdx.x], b = start[blockIdx.x + 1], tid = threadIdx.x;
    if (a == b) {
        if (tid == 0) count[blockIdx.x] = 0;
        return;
    }
    for (uint32_t s = tid; s < S; s += blockDim.x) {
        lk[s] = 0;
        lh[s] = kNobody;
    }
    if (tid == 0) n_out = n_many = full = 0;
    __syncthreads();
    for (uint32_t i = a + tid; i < b; i += blockDim.x) {
        const uint64_t y = key[i];
        const unsigned long long k = part_value(y, bits);
        const uint32_t d = dec[i];
        uint32_t s = (uint32_t)(y >> 32) / (0xFFFFFFFFu / S + 1u), probe = 0;   // the top bits after the part's
        auto take = [&]() {
            unsigned long long cur = *(volatile unsigned long long *)&lk[s];
            if (cur == 0) cur = atomicCAS(&lk[s], 0ull, k);
            return cur == 0 || cur == k;
        };
        bool placed = false;
        for (; probe < kShortProbe; ++probe, s = (s + 1) & (S - 1))
            if ((placed = take())) break;
        if (!placed) {
            // more distinct hashes than slots: the set is built whole instead
            // (long probes ask for it, so that the part ends soon)
            for (; probe < S && !*(volatile uint32_t *)&full; ++probe, s = (s + 1) & (S - 1))
                if ((placed = take())) break;
            if (!placed) {
                if (probe == S) {
                    full = 1;
                    atomicOr(flag, 2u);
                }
                break;
            }
        }
        uint32_t h = *(volatile uint32_t *)&lh[s];
        if (h == kNobody) h = atomicCAS(&lh[s], kNobody, d);
        if (h != kNobody && !(h & kManyHolders) && h != d) atomicOr(&lh[s], kManyHolders);
    }
    __syncthreads();
    for (uint32_t s = tid; s < S; s += blockDim.x) {   // (S is a multiple of the workgroup)
        const unsigned long long k = lk[s];
        const lmask out = ballot(k != 0), many = ballot(k != 0 && (lh[s] & kManyHolders));
        uint32_t base = 0;
        if (threadIdx.x % kWave == 0) {
            base = atomicAdd(&n_out, (uint32_t)__builtin_popcountll(out));
            if (many) atomicAdd(&n_many, (uint32_t)__builtin_popcountll(many));
        }
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        if (k != 0) {
            const uint32_t o = a + base + __builtin_amdgcn_mbcnt_hi((uint32_t)(out >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)out, 0u));
            okey[o] = k;
            ohold[o] = lh[s];
        }
    }
    __syncthreads();
    if (tid == 0) {
        count[blockIdx.x] = n_out;
        atomicAdd(cnt, (unsigned long long)n_out);
        if (n_many) atomicAdd(cnt + 1, (unsigned long long)n_many);
    }
}

// Shared hashes up to which the shared index is built: 48 to 96 bytes each, at
// most 64 MiB, a quarter of the last-level cache.
constexpr uint64_t kSharedMaxRows = 1ull << 20;

// Cuckoo insertion of distinct hashes into a block of the set (in LDS), or into the whole set.  A key
// goes to an empty slot of either candidate bucket (compare-and-swap 0 ->
// key); when all four slots are taken it displaces the key of a random slot by
// atomic exchange (a random walk: a fresh key picks either bucket, a displaced
// key its other bucket) and carries the displaced key on.  A key is always
// either in the set or carried by exactly one thread, so none is lost.
constexpr uint32_t kMaxKicks = 2048;

__device__ inline bool try_place(unsigned long long *bk, unsigned long long key) {
    for (int slot = 0; slot < 2; ++slot)
        if (atomicCAS(bk + slot, 0ull, key) == 0ull) return true;
    return false;
}

// Place the key of mixed value x in the block of 2^lg buckets `tab`; false
// when the walk did not end.
__device__ inline bool cuckoo_place(unsigned long long *tab, uint32_t lg, uint32_t shift, uint32_t in_block,
                                    unsigned long long x) {
    const uint32_t mask = (1u << lg) - 1u;
    uint32_t from = 0xFFFFFFFFu;   // bucket the carried key was displaced from
    uint32_t rnd = (uint32_t)(x >> 20);
    for (uint32_t kick = 0; kick < kMaxKicks; ++kick) {
        uint32_t b1, b2;
        buckets_of(unmix_hash(x), shift, in_block, b1, b2);
        b1 &= mask;
        b2 &= mask;
        if (try_place(tab + 2 * b1, x) || try_place(tab + 2 * b2, x)) return true;
        // displace from the bucket the key did not just leave; the walk's
        // choices come from the full-period 32-bit LCG of Knuth and Lewis
        // (multiplier 1664525, increment 1013904223; Press et al.,
        // Numerical Recipes, "quick and dirty" generator)
        rnd = rnd * 1664525u + 1013904223u;
        const uint32_t b = (b1 == from) ? b2 : (b2 == from) ? b1 : ((rnd >> 31) ? b2 : b1);
        const unsigned long long old = atomicExch(tab + 2 * b + ((rnd >> 30) & 1u), x);
        if (old == 0ull) return true;
        x = old;
        from = b;
    }
    return false;
}

// The slot of mixed value x in the block, or ~0.
__device__ inline uint32_t slot_of(const unsigned long long *tab, uint32_t lg, uint32_t shift, uint32_t in_block,
                                   unsigned long long x) {
    const uint32_t mask = (1u << lg) - 1u;
    uint32_t b1, b2;
    buckets_of(unmix_hash(x), shift, in_block, b1, b2);
    b1 &= mask;
    b2 &= mask;
    return tab[2 * b1] == x ? 2 * b1 : tab[2 * b1 + 1] == x ? 2 * b1 + 1
         : tab[2 * b2] == x ? 2 * b2 : tab[2 * b2 + 1] == x ? 2 * b2 + 1 : 0xFFFFFFFFu;
}

struct Build {
    const uint64_t *key;      // the pairs, by part (part_key)
    const uint32_t *dec;
    const uint64_t *dkey;     // the distinct hashes of each part
    const uint32_t *dhold;
    const uint32_t *start, *count;
    uint32_t bits;            // 2^bits parts
    uint32_t lg;              // 2^lg buckets per block, at most S / 2
    uint32_t log2b;           // 2^log2b buckets
    uint64_t *keys;           // the set
    uint32_t *vals;
    uint64_t *rows;           // bitmap rows, cleared; handed out from 1
    uint32_t bpitch;
    u32x4 *shared;            // shared index, cleared, or null
    uint32_t sh_shift, sh_mask;
    uint32_t *rows_used;
    uint32_t *flag;
};

// One workgroup per block of the set.  The block's hashes are those of one
// part, a piece of one, or of several.
template <uint32_t S>
__global__ __launch_bounds__(1024) void build_kernel(Build u) {
    __shared__ unsigned long long lk[S];
    __shared__ uint32_t lv[S];
    __shared__ uint32_t n_many, n_used, base;
    const uint32_t tid = threadIdx.x, shift = 64 - u.log2b, in_block = block_shift(shift), n_slot = 2u << u.lg;
    const uint64_t b0 = (uint64_t)blockIdx.x << u.lg;   // the block's first bucket
    const uint32_t p0 = u.log2b >= u.bits ? (uint32_t)(b0 >> (u.log2b - u.bits)) : (uint32_t)(b0 << (u.bits - u.log2b));
    const uint64_t b1 = b0 + (1ull << u.lg);
    const uint32_t p1 = u.log2b >= u.bits ? (uint32_t)((b1 - 1) >> (u.log2b - u.bits)) + 1
                                          : (uint32_t)(b1 << (u.bits - u.log2b));
    // f(position) over the pairs or the distinct hashes of the block's parts:
    // a wavefront per part where there are many, else all threads on each
    const uint32_t wv = wave_index(), nwv = blockDim.x / kWave, lane = tid % kWave;
    const bool spread = p1 - p0 < nwv;
    auto each = [&](bool pairs, auto f) {
        for (uint32_t p = spread ? p0 : p0 + wv; p < p1; p += spread ? 1 : nwv) {
            const uint32_t a = u.start[p], e = pairs ? u.start[p + 1] : a + u.count[p];
            for (uint32_t i = a + (spread ? tid : lane); i < e; i += spread ? blockDim.x : kWave) f(i);
        }
    };
    auto mine = [&](unsigned long long x) { return x >> shift >> u.lg == blockIdx.x; };
    for (uint32_t s = tid; s < n_slot; s += blockDim.x) {
        lk[s] = 0;
        lv[s] = 0;
    }
    if (tid == 0) n_many = n_used = 0;
    __syncthreads();
    each(false, [&](uint32_t i) {
        const unsigned long long x = u.dkey[i];
        if (!mine(x)) return;
        if (!cuckoo_place(lk, u.lg, shift, in_block, x)) atomicOr(u.flag, kErrTableFull);
        if (u.dhold[i] & kManyHolders) atomicAdd(&n_many, 1u);
    });
    __syncthreads();
    if (tid == 0) base = n_many ? atomicAdd(u.rows_used, n_many) : 0u;
    __syncthreads();
    each(false, [&](uint32_t i) {
        const unsigned long long x = u.dkey[i];
        if (!mine(x)) return;
        const uint32_t hold = u.dhold[i];
        uint32_t v = kHeldOne | hold;
        if (hold & kManyHolders) {
            v = base + atomicAdd(&n_used, 1u);
            if (u.shared) {
                // ends: there are more slots than keys
                const uint64_t h = unmix_hash(x);
                uint32_t j = (uint32_t)((h * kGolden) >> u.sh_shift);
                while (atomicCAS((unsigned long long *)(u.shared + j), 0ull, (unsigned long long)h) != 0ull)
                    j = (j + 1) & u.sh_mask;
                ((uint32_t *)(u.shared + j))[2] = v;
            }
        }
        const uint32_t s = slot_of(lk, u.lg, shift, in_block, x);
        if (s != 0xFFFFFFFFu) lv[s] = v;   // (else the walk failed, which was flagged)
    });
    __syncthreads();
    for (uint32_t s = tid; s < n_slot; s += blockDim.x) {
        u.keys[2 * b0 + s] = unmix_hash(lk[s]);
        u.vals[2 * b0 + s] = lv[s];
    }
    // the bitmaps: this workgroup alone writes its rows, so the atomics stay
    // in this die's cache
    if (n_many == 0) return;
    each(true, [&](uint32_t i) {
        const unsigned long long x = part_value(u.key[i], u.bits);
        if (!mine(x)) return;
        const uint32_t s = slot_of(lk, u.lg, shift, in_block, x);
        const uint32_t v = s != 0xFFFFFFFFu ? lv[s] : kHeldOne;
        if (v < kHeldOne) {
            const uint32_t d = u.dec[i];
            __hip_atomic_fetch_or(u.rows + (uint64_t)v * u.bpitch + d / 64u, 1ull << (d % 64u), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    });
}

// The whole set, built in memory from the pairs sorted by all bits of their
// keys, so that the holders of one hash form a run whose first element
// ("head") stands for it: the form of resident sets that the blocks cannot
// hold (five times the blocked build's time for 50.3 M pairs).
__device__ inline bool run_head(const uint64_t *__restrict__ key, uint64_t i) {
    return i == 0 || key[i] != key[i - 1];
}

// Least and largest holder of the run that starts at i, and its end.
__device__ inline uint64_t run_span(const uint64_t *__restrict__ key, const uint32_t *__restrict__ dec, uint64_t n,
                                    uint64_t i, uint32_t &dmin, uint32_t &dmax) {
    dmin = dmax = dec[i];
    uint64_t e = i + 1;
    for (; e < n && key[e] == key[i]; ++e) {
        dmin = min(dmin, dec[e]);
        dmax = max(dmax, dec[e]);
    }
    return e;
}

// cnt[0] += distinct hashes, cnt[1] += hashes with two or more holders.
__global__ __launch_bounds__(256) void whole_count_kernel(const uint64_t *__restrict__ key,
                                                          const uint32_t *__restrict__ dec, uint64_t n,
                                                          unsigned long long *__restrict__ cnt) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint32_t heads = 0, many = 0;
    for (; i < n; i += stride) {
        if (!run_head(key, i)) continue;
        uint32_t dmin, dmax;
        run_span(key, dec, n, i, dmin, dmax);
        ++heads;
        many += dmin != dmax ? 1u : 0u;
    }
    heads = wave_sum_u32(heads);
    many = wave_sum_u32(many);
    if ((threadIdx.x % kWave) == 0) {
        if (heads) atomicAdd(cnt, (unsigned long long)heads);
        if (many) atomicAdd(cnt + 1, (unsigned long long)many);
    }
}

__global__ __launch_bounds__(256) void whole_insert_kernel(Build u, uint64_t n) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint32_t shift = 64 - u.log2b;
    for (; i < n; i += stride)
        if (run_head(u.key, i) && !cuckoo_place((unsigned long long *)u.keys, u.log2b, shift, shift,
                                                part_value(u.key[i], u.bits)))
            atomicOr(u.flag, kErrTableFull);
}

// Holder values, once every key has its slot; each bitmap row is written by
// the one thread of its run.
__global__ __launch_bounds__(256) void whole_value_kernel(Build u, uint64_t n) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint32_t shift = 64 - u.log2b;
    for (; i < n; i += stride) {
        if (!run_head(u.key, i)) continue;
        uint32_t dmin, dmax;
        const uint64_t e = run_span(u.key, u.dec, n, i, dmin, dmax);
        uint32_t v = kHeldOne | dmin;
        if (dmin != dmax) {
            v = atomicAdd(u.rows_used, 1u);
            uint64_t *row = u.rows + (uint64_t)v * u.bpitch;
            for (uint64_t x = i; x < e; ++x) row[u.dec[x] / 64u] |= 1ull << (u.dec[x] % 64u);
        }
        const uint32_t s = slot_of((const unsigned long long *)u.keys, u.log2b, shift, shift,
                                   part_value(u.key[i], u.bits));
        if (s != 0xFFFFFFFFu) u.vals[s] = v;   // (else the walk failed, which was flagged)
    }
}

// The set's mixed values back to hashes, once nothing looks them up.
__global__ __launch_bounds__(256) void whole_unmix_kernel(uint64_t *__restrict__ keys, uint64_t n) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) keys[i] = unmix_hash(keys[i]);
}

__global__ void fill_u64_kernel(uint64_t *__restrict__ p, uint64_t n, uint64_t v) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

__global__ void fill_u32_kernel(uint32_t *__restrict__ p, uint64_t n, uint32_t v) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

// ------------------------------------------------------------------ snapshot checks

// Predictive congestion (Sec. VIII): one step of simple exponential
// smoothing of the congestion matrix towards an observation,
// c <- c + beta (obs - c), in fp32.  Both lie in [0, 1) and the result is
// their convex combination, rounded between them, so it stays in [0, 1).
// An observation outside [0, 1) or NaN leaves its entry unchanged and
// raises kErrObservation.
__device__ inline float smooth_one(float u, float o, float beta, bool &bad) {
    if (!(o >= 0.0f && o < 1.0f)) {
        bad = true;
        return u;
    }
    return fmaf(beta, o - u, u);
}

// VEC4: both arrays 16-byte aligned; four entries per thread and step,
// the n % 4 tail by the first threads.
template <bool VEC4>
__global__ __launch_bounds__(256) void smooth_kernel(float *__restrict__ util, const float *__restrict__ obs,
                                                     uint64_t n, float beta, uint32_t *__restrict__ err) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    bool bad = false;
    if (VEC4) {
        const uint64_t n4 = n / 4;
        for (uint64_t v = i; v < n4; v += stride) {
            const float4 o = ((const float4 *)obs)[v];
            float4 u = ((const float4 *)util)[v];
            u.x = smooth_one(u.x, o.x, beta, bad);
            u.y = smooth_one(u.y, o.y, beta, bad);
            u.z = smooth_one(u.z, o.z, beta, bad);
            u.w = smooth_one(u.w, o.w, beta, bad);
            ((float4 *)util)[v] = u;
        }
        i += n4 * 4;
        if (i >= n4 * 4 + 4) i = n;   // only the first threads take the tail
    }
    for (; i < n; i += stride) util[i] = smooth_one(util[i], obs[i], beta, bad);
    if (__ballot(bad) && (threadIdx.x % kWave) == 0) atomicOr(err, kErrObservation);
}

// A snapshot whose arrays all lie in this device's memory is copied and
// checked in one pass (six copies, a clear and the check as launches of
// their own took about 45 us).
struct SnapIn {
    const uint8_t *tier;
    const float *util;
    const uint16_t *n_inflight;
    const uint64_t *free_mem;
    const uint32_t *queue, *batch;
};

__global__ __launch_bounds__(256) void load_snapshot_kernel(SnapIn in, uint64_t npd, uint32_t P, uint32_t D,
                                                            uint32_t beta_max, uint8_t *__restrict__ tier,
                                                            float *__restrict__ util,
                                                            uint16_t *__restrict__ n_inflight,
                                                            uint64_t *__restrict__ free_mem,
                                                            uint64_t *__restrict__ adm_prev,
                                                            uint32_t *__restrict__ queue,
                                                            uint32_t *__restrict__ batch,
                                                            uint32_t *__restrict__ bad) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint32_t f = 0;
    for (uint64_t x = i; x < npd; x += stride) {
        const uint8_t t = in.tier[x];
        const float u = in.util[x];
        if (t > 3) f |= 1u;
        if (!(u >= 0.0f && u < 1.0f)) f |= 2u;
        tier[x] = t;
        util[x] = u;
    }
    for (uint64_t x = i; x < 4ull * P; x += stride) n_inflight[x] = in.n_inflight[x];
    for (uint64_t x = i; x < D; x += stride) {
        const uint32_t b = in.batch[x];
        if (b > beta_max) f |= 4u;
        batch[x] = b;
        queue[x] = in.queue[x];
        free_mem[x] = in.free_mem[x];
        adm_prev[x] = 0;
    }
    if (f) atomicOr(bad, f);
}

__global__ void check_snapshot_kernel(const uint8_t *__restrict__ tier, const float *__restrict__ util,
                                      uint64_t npd, const uint32_t *__restrict__ batch, uint32_t D,
                                      uint32_t beta_max, uint32_t *__restrict__ bad) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint32_t f = 0;
    for (uint64_t x = i; x < npd; x += stride) {
        if (tier && tier[x] > 3) f |= 1u;
        float u = util[x];
        if (!(u >= 0.0f && u < 1.0f)) f |= 2u;
    }
    if (batch)
        for (uint64_t x = i; x < D; x += stride)
            if (batch[x] > beta_max) f |= 4u;
    if (f) atomicOr(bad, f);
}

// ------------------------------------------------------------------ between-batch update

// First-miss scan of one (hash run, decode) pair by one thread.
__device__ inline uint32_t prefix_match_one(const Table &t, uint32_t d, const uint64_t *__restrict__ run,
                                            uint32_t n) {
    uint32_t j = 0;
    while (j < n && holds(t, run[j], d)) ++j;
    return j;
}

// The same by kMatchLanes neighbouring lanes, a block each per step: a lookup
// is a chain of three dependent loads (buckets, holder value, bitmap word),
// and one thread walking a run of a hundred resident blocks keeps its
// workgroup waiting for 100 us.  Every lane of the wavefront must call it;
// n = 0 for those without a request.  All lanes of a group get the result.
constexpr uint32_t kMatchLanes = 16;
__device__ inline uint32_t prefix_match_lanes(const Table &t, uint32_t d, const uint64_t *__restrict__ run,
                                              uint32_t n) {
    const uint32_t sub = threadIdx.x % kMatchLanes, seg0 = (threadIdx.x % kWave) - sub;
    uint32_t j = n;
    bool act = n > 0;
    for (uint32_t k0 = 0; __any(act); k0 += kMatchLanes) {
        const uint32_t k = k0 + sub;
        const bool miss = act && (k >= n || !holds(t, run[k], d));
        const uint32_t m = (uint32_t)(__ballot(miss) >> seg0) & ((1u << kMatchLanes) - 1u);
        if (act && m) {
            j = k0 + (uint32_t)__builtin_ctz(m);
            act = false;
        }
    }
    return j;
}

__global__ void commit_count_kernel(Snap s, Table t, Reqs rq, const int32_t *__restrict__ sel,
                                    uint32_t *__restrict__ cnt, uint32_t *__restrict__ adm,
                                    unsigned long long *__restrict__ bytes, uint32_t *__restrict__ err) {
    uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rq.n_req) return;
    int32_t d = sel[r];
    if (d < 0) return;
    if ((uint32_t)d >= s.D) {
        atomicOr(err, kErrSelection);
        return;
    }
    uint32_t p, len, n;
    uint64_t a;
    if (!request_ok(rq, s, r, p, len, a, n)) {
        atomicOr(err, kErrRequest);
        return;
    }
    uint32_t j = prefix_match_one(t, (uint32_t)d, rq.hashes + a, n);
    uint64_t s_eff = (uint64_t)s.bpt * (uint64_t)(len - s.block_tokens * j);
    uint32_t tau = s.tier_map[(uint64_t)p * s.D + (uint32_t)d] & 3u;
    atomicAdd(cnt + tau * s.P + p, 1u);
    atomicAdd(adm + d, 1u);
    atomicAdd(bytes + d, (unsigned long long)s_eff);
}

// Between-batch update of one counter entry i (of 4 P in-flight counters,
// then D decodes) from the batch's sums.
__device__ inline void commit_entry(uint32_t i, uint32_t P, uint32_t cap, uint32_t mu, uint32_t c,
                                    unsigned long long b, uint16_t *__restrict__ n_inflight,
                                    uint32_t *__restrict__ queue, uint64_t *__restrict__ free_mem,
                                    uint64_t *__restrict__ adm_prev) {
    if (i < 4 * P) {
        n_inflight[i] = (uint16_t)(c < cap ? c : cap);
        return;
    }
    const uint32_t d = i - 4 * P;
    const int64_t nq = (int64_t)queue[d] + (int64_t)c - (int64_t)mu;
    queue[d] = (uint32_t)(nq < 0 ? 0 : nq);
    uint64_t m = free_mem[d];
    m = m > b ? m - b : 0;
    free_mem[d] = m + adm_prev[d];
    adm_prev[d] = b;
}

__global__ void commit_apply_kernel(uint32_t P, uint32_t D, uint32_t cap, uint32_t mu,
                                    const uint32_t *__restrict__ cnt, const uint32_t *__restrict__ adm,
                                    const unsigned long long *__restrict__ bytes,
                                    uint16_t *__restrict__ n_inflight, uint32_t *__restrict__ queue,
                                    uint64_t *__restrict__ free_mem, uint64_t *__restrict__ adm_prev) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 4 * P + D) return;
    const uint32_t d = i - 4 * P;
    commit_entry(i, P, cap, mu, i < 4 * P ? cnt[i] : adm[d], i < 4 * P ? 0ull : bytes[d], n_inflight, queue, free_mem,
                 adm_prev);
}

// The same sums without device-wide atomics: a batch puts R / (4 P) and
// R / D requests on each counter, and same-address atomics of all
// workgroups are served one after another (245 us for 65,536 requests on
// 16 x 48 instances, 0.18 us per atomic of one address).  Each workgroup
// sums its requests in LDS (cnt[4 P], adm[D], bytes[D]) and writes its sums
// to its own row; commit_sum_kernel adds the rows.
constexpr uint32_t kCommitThreads = 1024;
constexpr uint32_t kCommitRows = 256;             // most workgroups (rows)
constexpr uint64_t kCommitLds = 64ull << 10;      // LDS of one workgroup's sums

__global__ __launch_bounds__(kCommitThreads) void commit_rows_kernel(Snap s, Table t, Reqs rq,
                                                                     const int32_t *__restrict__ sel,
                                                                     uint32_t *__restrict__ rows,
                                                                     unsigned long long *__restrict__ brows,
                                                                     uint32_t *__restrict__ err) {
    extern __shared__ unsigned long long csum[];   // bytes[D], then counts [4 P + D]
    uint32_t *cnt = (uint32_t *)(csum + s.D);
    const uint32_t n = 4 * s.P + s.D;
    for (uint32_t i = threadIdx.x; i < s.D; i += kCommitThreads) csum[i] = 0;
    for (uint32_t i = threadIdx.x; i < n; i += kCommitThreads) cnt[i] = 0;
    __syncthreads();
    uint32_t bad = 0;
    constexpr uint32_t kPer = kCommitThreads / kMatchLanes;   // requests per workgroup and step
    const bool head = threadIdx.x % kMatchLanes == 0;
    for (uint64_t r0 = (uint64_t)blockIdx.x * kPer; r0 < rq.n_req; r0 += (uint64_t)gridDim.x * kPer) {
        const uint64_t r = r0 + threadIdx.x / kMatchLanes;
        int32_t d = r < rq.n_req ? sel[r] : -1;
        uint32_t p = 0, len = 0, nb = 0;
        uint64_t a = 0;
        if (d >= 0 && (uint32_t)d >= s.D) {
            bad |= kErrSelection;
            d = -1;
        }
        if (d >= 0 && !request_ok(rq, s, (uint32_t)r, p, len, a, nb)) {
            bad |= kErrRequest;
            d = -1;
        }
        const uint32_t j = prefix_match_lanes(t, (uint32_t)d, rq.hashes + a, d < 0 ? 0u : nb);
        if (d >= 0 && head) {
            const uint32_t tau = s.tier_map[(uint64_t)p * s.D + (uint32_t)d] & 3u;
            atomicAdd(cnt + tau * s.P + p, 1u);
            atomicAdd(cnt + 4 * s.P + (uint32_t)d, 1u);
            atomicAdd(csum + d, (unsigned long long)((uint64_t)s.bpt * (uint64_t)(len - s.block_tokens * j)));
        }
    }
    if (bad) atomicOr(err, bad);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += kCommitThreads) rows[(uint64_t)blockIdx.x * n + i] = cnt[i];
    for (uint32_t i = threadIdx.x; i < s.D; i += kCommitThreads) brows[(uint64_t)blockIdx.x * s.D + i] = csum[i];
}

// One wavefront per counter entry: the sum over the rows, then the update.
__global__ __launch_bounds__(256) void commit_sum_kernel(uint32_t P, uint32_t D, uint32_t cap, uint32_t mu,
                                                         uint32_t nrow, const uint32_t *__restrict__ rows,
                                                         const unsigned long long *__restrict__ brows,
                                                         uint16_t *__restrict__ n_inflight,
                                                         uint32_t *__restrict__ queue,
                                                         uint64_t *__restrict__ free_mem,
                                                         uint64_t *__restrict__ adm_prev) {
    const uint32_t n = 4 * P + D;
    const uint32_t i = blockIdx.x * kWavesPerBlock + wave_index(), lane = threadIdx.x % kWave;
    if (i >= n) return;
    uint32_t c = 0;
    unsigned long long b = 0;
    for (uint32_t w = lane; w < nrow; w += kWave) {
        c += rows[(uint64_t)w * n + i];
        if (i >= 4 * P) b += brows[(uint64_t)w * D + (i - 4 * P)];
    }
    c = wave_sum_u32(c);
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) b += __shfl_xor(b, m, kWave);
    if (lane == 0) commit_entry(i, P, cap, mu, c, b, n_inflight, queue, free_mem, adm_prev);
}

// ---------------------------------------------------------------- tier counts

// Two-hop routing: the route each selection takes (1: staged, 0: direct,
// -1: no selection or an invalid request): the selected pair's prefix
// length (first miss of the run on that decode), then its direct and
// staged costs from the derived rows, in the scoring kernel's arithmetic.
__global__ __launch_bounds__(256) void route_of_kernel(Snap s, Table t, Reqs rq, uint32_t k,
                                                       const int32_t *__restrict__ idx, int8_t *__restrict__ out) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (uint64_t)rq.n_req * k) return;
    const uint32_t r = (uint32_t)(i / k);
    const int32_t d = idx[i];
    uint32_t p, len, n;
    uint64_t a;
    if (d < 0 || (uint32_t)d >= s.D || !request_ok(rq, s, r, p, len, a, n)) {
        out[i] = -1;
        return;
    }
    uint32_t j = 0;
    while (j < n && holds(t, rq.hashes[a + j], (uint32_t)d)) ++j;
    const float x = (float)(len - s.block_tokens * j);
    const uint64_t o = (uint64_t)p * s.slp + (uint32_t)d;
    const float2 r1 = s.sl[o], r2 = s.sr[o];
    out[i] = fmaf(x, r2.x, r2.y) < fmaf(x, r1.x, r1.y) ? 1 : 0;
}

// Non-cached bytes of each selection (Eq. (2) in the integer form
// bpt * (l_r - B_tok * j)): the selected pair's prefix length by the first
// miss of the run on that decode.  0 for no selection or an invalid
// request; a selection index >= D is flagged.
__global__ __launch_bounds__(256) void selection_bytes_kernel(Snap s, Table t, Reqs rq, uint32_t k,
                                                              const int32_t *__restrict__ idx,
                                                              uint64_t *__restrict__ out, uint32_t *__restrict__ err) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (uint64_t)rq.n_req * k) return;
    const uint32_t r = (uint32_t)(i / k);
    const int32_t d = idx[i];
    uint32_t p, len, n;
    uint64_t a;
    if (d >= 0 && (uint32_t)d >= s.D) atomicOr(err, kErrSelection);
    if (d < 0 || (uint32_t)d >= s.D || !request_ok(rq, s, r, p, len, a, n)) {
        out[i] = 0;
        return;
    }
    uint32_t j = 0;
    while (j < n && holds(t, rq.hashes[a + j], (uint32_t)d)) ++j;
    out[i] = (uint64_t)s.bpt * (uint64_t)(len - s.block_tokens * j);
}

// Requests per tier of the selected decode (index 4: rejected), the tier
// shift statistic.  Invalid selections are flagged and not counted.
__global__ __launch_bounds__(256) void tier_count_kernel(Snap s, Reqs rq, const int32_t *__restrict__ sel,
                                                         unsigned long long *__restrict__ counts,
                                                         uint32_t *__restrict__ err) {
    __shared__ uint32_t local[5];
    if (threadIdx.x < 5) local[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < rq.n_req) {
        const int32_t d = sel[r];
        const uint32_t p = rq.prefill[r];
        if (d < 0) {
            atomicAdd(&local[4], 1u);
        } else if ((uint32_t)d < s.D && p < s.P) {
            atomicAdd(&local[s.tier_map[(uint64_t)p * s.D + (uint32_t)d] & 3u], 1u);
        } else {
            atomicOr(err, kErrSelection);
        }
    }
    __syncthreads();
    if (threadIdx.x < 5 && local[threadIdx.x]) atomicAdd(counts + threadIdx.x, (unsigned long long)local[threadIdx.x]);
}

// ---------------------------------------------------------------- sequential selection
//
// Algorithm 1 applied request after request in batch order: the in-flight
// counter of the chosen tier grows by one (up to the cap) before the next
// request from the same prefill instance is scored.  Requests of different
// prefill instances do not interact, so each prefill instance's requests are
// a sequential chain run by one workgroup.  The prefix lengths come from the
// batch selection's scoring records (by batch index) and leader rows: the
// chain reads min(leader row, B_tok * L*) per decode, as the scoring kernel
// does, and no per-pair buffer is written.

// start/end of each prefill instance's run in the order sorted by prefill
__global__ void segment_kernel(const uint32_t *__restrict__ keys, uint32_t n, uint32_t P, uint32_t *__restrict__ start,
                               uint32_t *__restrict__ end) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t k = keys[i];
    if (k >= P) return;
    if (i == 0 || keys[i - 1] != k) start[k] = i;
    if (i + 1 == n || keys[i + 1] != k) end[k] = i + 1;
}

// (an invalid request's record has length 0)
__global__ void prefill_key_kernel(Reqs rq, uint32_t P, const Hot *__restrict__ hotr,
                                   uint32_t *__restrict__ keys, uint32_t *__restrict__ vals) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rq.n_req) return;
    keys[r] = hotr[r].len == 0 ? P : rq.prefill[r];
    if (vals) vals[r] = r;
}

// Non-cached tokens x (Eq. (2)) of request r on decodes d0 + stride * k,
// k < M, from its scoring record: the leader row capped by B_tok * L*, or,
// for a request marked to match on its own, a first-miss scan of its hash
// run over the holder index.  Integers throughout (a record's fp32 values
// are integers below 2^24, so exact).  Decodes at or past D get len; the
// caller never finds them feasible.
template <int M>
__device__ inline void seq_tokens(const Snap &s, const Table &t, const Reqs &rq, const Hot *__restrict__ hotr,
                                  const float *__restrict__ lead_lam, uint32_t r, uint32_t d0, uint32_t stride,
                                  uint32_t (&x)[M]) {
    const Hot rec = hotr[r];
    if ((int32_t)rec.lams >= 0) {
        const uint32_t len = (uint32_t)__uint_as_float(rec.len);
        const float *row = lead_lam + rec.lrow / sizeof(float);
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const uint32_t d = d0 + stride * k;
            const uint32_t lam = d < s.D ? min(__float_as_uint(row[d]), rec.lams) : 0u;
            x[k] = len - (uint32_t)__uint_as_float(lam);
        }
        return;
    }
    uint32_t p, len, n;
    uint64_t a;
    request_ok(rq, s, r, p, len, a, n);   // validated by the selection
    uint32_t j[M];
    uint32_t alive = 0;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        j[k] = n;
        alive |= (d0 + stride * k < s.D ? 1u : 0u) << k;
    }
    for (uint32_t b = 0; b < n && alive; ++b) {
        const uint32_t v = holder_lane(t, rq.hashes[a + b]);
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const uint32_t d = d0 + stride * k;
            if (((alive >> k) & 1u) && !((held_mask(t, v, d & ~(uint32_t)(kWave - 1)) >> (d % kWave)) & 1ull)) {
                j[k] = b;
                alive &= ~(1u << k);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < M; ++k) x[k] = len - s.block_tokens * j[k];
}

constexpr int kSeqThreads = 256;

constexpr int kSeqChunk = 8;   // decodes per thread per pass of the general chain

__global__ __launch_bounds__(kSeqThreads) void sequential_kernel(Snap s, Table t, Reqs rq, uint32_t cap,
                                                                 const Hot *__restrict__ hotr,
                                                                 const float *__restrict__ lead_lam,
                                                                 const uint32_t *__restrict__ order,
                                                                 const uint32_t *__restrict__ start,
                                                                 const uint32_t *__restrict__ end,
                                                                 int32_t *__restrict__ out_idx,
                                                                 float *__restrict__ out_score) {
    __shared__ float n_tier[4];
    __shared__ uint32_t best_cost[kSeqThreads / kWave];
    __shared__ uint32_t best_d[kSeqThreads / kWave];
    const uint32_t p = blockIdx.x;
    const uint32_t i0 = start[p], i1 = end[p];
    if (i0 >= i1) return;
    const uint32_t lane = threadIdx.x % kWave, wave = wave_index();
    if (threadIdx.x < 4) n_tier[threadIdx.x] = (float)s.n_inflight[threadIdx.x * s.P + p];
    __syncthreads();
    for (uint32_t i = i0; i < i1; ++i) {
        const uint32_t r = order[i];
        uint32_t lb = 0xFFFFFFFFu, ld = 0xFFFFFFFFu;
        for (uint32_t d0 = threadIdx.x; d0 < s.D; d0 += kSeqThreads * kSeqChunk) {
            uint32_t xc[kSeqChunk];
            seq_tokens<kSeqChunk>(s, t, rq, hotr, lead_lam, r, d0, kSeqThreads, xc);
#pragma unroll
            for (int k = 0; k < kSeqChunk; ++k) {
                const uint32_t d = d0 + kSeqThreads * k, x = xc[k];
                if (d < s.D && (uint64_t)x < s.dxlim[d]) {
                    const uint64_t o = (uint64_t)p * s.D + d;
                    const uint32_t tau = s.tier_map[o] & 3u;
                    const float cost = pair_score(x, sec_per_token_n(s, tau, n_tier[tau], s.util[o]), s.lat[tau],
                                                  s.dbase[d]);
                    const uint32_t cbits = __float_as_uint(cost);
                    if (cbits < lb) {   // d grows within a thread: first strict minimum wins ties
                        lb = cbits;
                        ld = d;
                    }
                }
            }
        }
        const uint32_t mn = wave_min_u32_dpp(lb);
        const uint32_t dm = wave_min_u32_dpp(lb == mn ? ld : 0xFFFFFFFFu);
        if (lane == 0) {
            best_cost[wave] = mn;
            best_d[wave] = dm;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t bc = best_cost[0], bd = best_d[0];
            for (int w = 1; w < kSeqThreads / kWave; ++w)
                if (best_cost[w] < bc || (best_cost[w] == bc && best_d[w] < bd)) {
                    bc = best_cost[w];
                    bd = best_d[w];
                }
            if (bc == 0xFFFFFFFFu) {
                out_idx[r] = -1;
                out_score[r] = __builtin_inff();
            } else {
                out_idx[r] = (int32_t)bd;
                out_score[r] = __uint_as_float(bc);
                const uint32_t tau = s.tier_map[(uint64_t)p * s.D + bd] & 3u;
                if (n_tier[tau] < (float)cap) n_tier[tau] += 1.0f;
            }
        }
        __syncthreads();
    }
}

// One of four uniform values by a per-lane index, without indexing an array.
__device__ inline float pick4(const float (&v)[4], uint32_t t) {
    const float lo = (t & 1u) ? v[1] : v[0];
    const float hi = (t & 1u) ? v[3] : v[2];
    return (t & 2u) ? hi : lo;
}

// The same chain with each thread's decodes (d = thread + T*k, k < MAXC)
// held in registers: tier (2 bits each in one word), seconds per token,
// tier latency plus load term, and the feasibility limit (32 bits, with a
// bit for limits of 2^32 and more, which every x meets); the prefill row's
// congestion sits in LDS.  Between requests only the factors of the tier
// whose counter grew change, and they are recomputed with the same
// expression.
//
// Pipeline: the chain's scoring records (and batch indices) are staged in
// LDS T at a time, two chunks deep, so a request's record is an LDS read;
// the leader-row values of the next request are loaded while the current
// one is scored (raw bits, into the other of two buffers).  Each wave's
// minimum carries the winner's decode and tier (d << 2 | tier), the waves'
// minima go to alternating LDS slots and every thread picks the winner, so
// one barrier per request suffices (a wave can write a slot again only
// after the barrier that follows every wave's reading of it) and the
// counter update needs no memory read.
template <int MAXC>
struct SeqBuf {
    uint32_t raw[MAXC];   // leader-row bits B_tok * j, or B_tok * j itself (own scan)
    uint32_t len, lams, own, r;
};

template <int T, int MAXC>
__global__ __launch_bounds__(T, MAXC <= 12 ? 4 : 1) void sequential_cached_kernel(Snap s, Table t, Reqs rq, uint32_t cap,
                                                              const Hot *__restrict__ hotr,
                                                              const float *__restrict__ lead_lam,
                                                              const uint32_t *__restrict__ order,
                                                              const uint32_t *__restrict__ start,
                                                              const uint32_t *__restrict__ end,
                                                              int32_t *__restrict__ out_idx,
                                                              float *__restrict__ out_score) {
    static_assert(MAXC <= 16, "two tier bits per decode in one word");
    constexpr int NW = T / kWave;
    __shared__ uint32_t slot_c[2][NW], slot_d[2][NW];
    __shared__ Hot crec[2][T];
    __shared__ uint32_t cr[2][T];
    // per thread-decode (index k * T + thread), each entry only ever used by
    // its own thread: the congestion, and a staging area for seconds per
    // token (set-up, counter updates) or an own scan's B_tok * j
    __shared__ float urow[T * MAXC];
    __shared__ uint32_t stage[T * MAXC];
    const uint32_t p = blockIdx.x;
    const uint32_t i0 = start[p], i1 = end[p];
    if (i0 >= i1) return;
    const uint32_t lane = threadIdx.x % kWave, wave = wave_index();
    const uint64_t row = (uint64_t)p * s.D;
    float n_tier[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) n_tier[q] = (float)s.n_inflight[q * s.P + p];
    uint32_t tmask = 0;
    float sk[MAXC], lk[MAXC], xm[MAXC];
    // the factors, one decode at a time through LDS (keeps the divisions'
    // temporaries out of the register budget)
#pragma unroll 1
    for (int k = 0; k < MAXC; ++k) {
        const uint32_t d = threadIdx.x + T * k;
        const uint32_t dd = d < s.D ? d : 0;
        const uint32_t tq = s.tier_map[row + dd] & 3u;
        const float u = s.util[row + dd];
        urow[k * T + threadIdx.x] = u;
        stage[k * T + threadIdx.x] = __float_as_uint(sec_per_token_n(s, tq, pick4(n_tier, tq), u));
        tmask |= tq << (2 * k);
    }
#pragma unroll
    for (int k = 0; k < MAXC; ++k) {
        const uint32_t d = threadIdx.x + T * k;
        const bool ok = d < s.D;
        const uint32_t dd = ok ? d : 0;
        sk[k] = __uint_as_float(stage[k * T + threadIdx.x]);
        lk[k] = tier_latency(s, (tmask >> (2 * k)) & 3u) + s.dbase[dd];
        // the largest feasible token count, as fp32 (exact: capped at 2^24,
        // beyond every count of the fp32 path); -1 when nothing is feasible
        // (and for decodes past D, never chosen)
        const uint64_t xl = ok ? s.dxlim[dd] : 0;
        xm[k] = xl == 0 ? -1.0f : (float)(xl - 1 < kExactTok ? xl - 1 : (uint64_t)kExactTok);
    }
    // stage chunk c (positions i0 + c*T ...) of the chain's records in LDS
    auto fill = [&](uint32_t c) {
        const uint32_t i = i0 + c * T + threadIdx.x;
        if (i < i1) {
            const uint32_t r = order[i];
            crec[c & 1u][threadIdx.x] = hotr[r];
            cr[c & 1u][threadIdx.x] = r;
        }
    };
    // read position i's record and start loading its leader-row values
    auto issue = [&](uint32_t i, SeqBuf<MAXC> &b) {
        const uint32_t o = i - i0, c = o / T;
        if (o % T == 0 && c >= 1) fill(c + 1);   // chunk c-1's last record was read before the last barrier
        const Hot &h = crec[c & 1u][o % T];
        const uint32_t r = __builtin_amdgcn_readfirstlane(cr[c & 1u][o % T]);
        const uint32_t lams = __builtin_amdgcn_readfirstlane(h.lams);
        b.r = r;
        if ((int32_t)lams >= 0) {
            const float *lrow = lead_lam + __builtin_amdgcn_readfirstlane(h.lrow) / sizeof(float);
            b.len = (uint32_t)__uint_as_float(__builtin_amdgcn_readfirstlane(h.len));
            b.lams = lams;
            b.own = 0;
#pragma unroll
            for (int k = 0; k < MAXC; ++k) {
                // decodes past D read decode 0's value; their limit 0 makes them infeasible
                const uint32_t d = threadIdx.x + T * k;
                b.raw[k] = __float_as_uint(lrow[d < s.D ? d : 0u]);
            }
        } else {
            // matched on its own: a first-miss scan of its run per decode, in
            // integers, B_tok * j through LDS
            uint32_t pp, len, n;
            uint64_t a;
            request_ok(rq, s, r, pp, len, a, n);   // validated by the selection
#pragma unroll 1
            for (int k = 0; k < MAXC; ++k) {
                const uint32_t d = threadIdx.x + T * k;
                uint32_t j = n;
                if (d < s.D) {
                    const uint32_t db = d & ~(uint32_t)(kWave - 1), bit = d % kWave;
                    for (uint32_t bk = 0; bk < n; ++bk)
                        if (!((held_mask(t, holder_lane(t, rq.hashes[a + bk]), db) >> bit) & 1ull)) {
                            j = bk;
                            break;
                        }
                }
                stage[k * T + threadIdx.x] = s.block_tokens * j;
            }
            b.len = len;
            b.lams = 0xFFFFFFFFu;
            b.own = 1;
#pragma unroll
            for (int k = 0; k < MAXC; ++k) b.raw[k] = stage[k * T + threadIdx.x];
        }
    };
    // score the buffered request, choose, count the choice
    auto step = [&](uint32_t i, const SeqBuf<MAXC> &b) {
        // the lane's least cost bits and the k of its decode: from the leader
        // row in fp32 (token counts below 2^24 are exact, as in the scoring
        // kernel), or for a request matched on its own in integers
        uint32_t lb = 0xFFFFFFFFu, kf = 0;
        if (!b.own) {
            const float lenf = (float)b.len;
#pragma unroll
            for (int k = 0; k < MAXC; ++k) {
                const float x = lenf - __uint_as_float(min(b.raw[k], b.lams));
                const uint32_t c = __float_as_uint(fmaf(x, sk[k], lk[k]));
                if (x <= xm[k] && c < lb) {   // d grows with k: the first strict minimum wins ties
                    lb = c;
                    kf = (uint32_t)k;
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < MAXC; ++k) {
                const uint32_t d = threadIdx.x + T * k;
                const uint32_t x = b.len - b.raw[k];
                if (d < s.D && (uint64_t)x < s.dxlim[d < s.D ? d : 0]) {
                    const uint32_t c = __float_as_uint(fmaf((float)x, sk[k], lk[k]));
                    if (c < lb) {
                        lb = c;
                        kf = (uint32_t)k;
                    }
                }
            }
        }
        const uint32_t ld = lb == 0xFFFFFFFFu ? 0xFFFFFFFFu
                                              : ((threadIdx.x + T * kf) << 2) | ((tmask >> (2 * kf)) & 3u);
        const uint32_t mn = wave_min_u32_dpp(lb);
        const uint32_t dm = wave_min_u32_dpp(lb == mn ? ld : 0xFFFFFFFFu);
        const uint32_t sl = i & 1u;
        if (lane == 0) {
            slot_c[sl][wave] = mn;
            slot_d[sl][wave] = dm;
        }
        __syncthreads();
        uint32_t bc = slot_c[sl][0], bd = slot_d[sl][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            const uint32_t c = slot_c[sl][w], dw = slot_d[sl][w];
            if (c < bc || (c == bc && dw < bd)) {
                bc = c;
                bd = dw;
            }
        }
        if (threadIdx.x == 0) {
            out_idx[b.r] = bc == 0xFFFFFFFFu ? -1 : (int32_t)(bd >> 2);
            out_score[b.r] = bc == 0xFFFFFFFFu ? __builtin_inff() : __uint_as_float(bc);
        }
        if (bc != 0xFFFFFFFFu) {
            const uint32_t tw = bd & 3u;
            const float nw = pick4(n_tier, tw);
            if (nw < (float)cap) {
                // at most cap times per tier: the tier's factors again, with
                // the same expression, through LDS
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((uint32_t)q == tw) n_tier[q] = nw + 1.0f;
#pragma unroll
                for (int k = 0; k < MAXC; ++k) stage[k * T + threadIdx.x] = __float_as_uint(sk[k]);
#pragma unroll 1
                for (int k = 0; k < MAXC; ++k)
                    if (((tmask >> (2 * k)) & 3u) == tw)
                        stage[k * T + threadIdx.x] =
                            __float_as_uint(sec_per_token_n(s, tw, nw + 1.0f, urow[k * T + threadIdx.x]));
#pragma unroll
                for (int k = 0; k < MAXC; ++k) sk[k] = __uint_as_float(stage[k * T + threadIdx.x]);
            }
        }
    };
    fill(0);
    fill(1);
    __syncthreads();
    SeqBuf<MAXC> ba, bb;
    issue(i0, ba);
    for (uint32_t i = i0; i < i1; i += 2) {
        if (i + 1 < i1) issue(i + 1, bb);
        step(i, ba);
        if (i + 1 >= i1) break;
        if (i + 2 < i1) issue(i + 2, ba);
        step(i + 1, bb);
    }
}

// Work buffers of one selection: per-request ordering buffers and records,
// the leader table, the leaders' holder values, per-group partial top-k
// keys and the sort / scan temporaries.  Owned by the handle (grown on
// demand, or sized ahead by netkv_reserve) or carved from the library's
// static scratch array (netkv_select_batch_noalloc).
struct Scratch {
    uint64_t order_cap = 0;   // requests the per-request buffers hold
    uint32_t *keys_in = nullptr, *keys_out = nullptr, *vals_in = nullptr, *perm = nullptr;
    Hot *hot = nullptr;       // [order_cap + kHotPad] scoring-order records, the part every step reads
    Cold *cold = nullptr;     // and the request's index in the batch
    uint64_t *seg = nullptr;    // in-tile inclusive scan of the positions' (leader, L) elements, hash order
    uint64_t *tpre = nullptr;   // per order tile: its total, then the exclusive prefix of the tiles before it
    Pre *hrec = nullptr;      // prefill row and length by hash-order position
    Cold *crec = nullptr;
    uint32_t *pkey = nullptr, *pkey_out = nullptr, *pval = nullptr, *pord = nullptr;   // prefill order
    uint32_t *n_valid = nullptr;
    unsigned long long *hv_used = nullptr;
    unsigned int *n_lead = nullptr;
    uint32_t *hv = nullptr;   // holder values of the leaders' blocks
    uint64_t hv_cap = 0;
    Lead *lead = nullptr;     // leader table
    float *lead_lam = nullptr;   // [lead_cap + 1][D] B_tok * prefix length of each leader;
                                 // row lead_cap is all zero (no leader)
    uint32_t lead_cap = 0, lead_D = 0;
    bool zero_row_set = false;   // row lead_cap has been cleared
    void *sort_tmp = nullptr;    // rocPRIM sort / scan temporary storage
    size_t sort_tmp_bytes = 0;
    // the batch sorts' own buffers: digit counts, totals and the ping-pong
    // pair (null when the per-request buffers hold no more than kSortMinN)
    uint32_t *sort_cnt = nullptr, *sort_tot = nullptr, *keys_tmp = nullptr, *vals_tmp = nullptr;
    uint64_t *partial = nullptr;   // [groups][R][K] per-group top-k keys
    uint64_t partial_cap = 0;
    Hot *hotr = nullptr;           // scoring records by batch index (ranking sweep, sequential form)
    uint64_t hotr_cap = 0;
};

}  // namespace

// ====================================================================== host side

// bytes of a cache load's work buffer that a handle keeps (89 M resident hashes)
constexpr uint64_t kLoadKeep = 2ull << 30;
constexpr uint32_t kTimeSlots = 256;   // timed launches kept for netkv_kernel_ms

struct netkv_ctx {
    int device = 0;
    std::string err;
    // snapshot
    bool have_snap = false;
    uint32_t P = 0, D = 0;
    uint8_t *tier_map = nullptr;
    float *util = nullptr;
    uint16_t *n_inflight = nullptr;
    uint64_t *free_mem = nullptr;
    uint32_t *queue = nullptr;
    uint32_t *batch = nullptr;
    uint64_t *adm_prev = nullptr;
    // the snapshot buffers of the load before, of the same shape: the next
    // load is staged and checked there, then the two are exchanged (a load
    // that allocated and freed its seven buffers spent about 150 us on it)
    struct SnapBuf {
        uint32_t P = 0, D = 0;   // shape; 0: no buffers
        uint8_t *tier_map = nullptr;
        float *util = nullptr;
        uint16_t *n_inflight = nullptr;
        uint64_t *free_mem = nullptr, *adm_prev = nullptr;
        uint32_t *queue = nullptr, *batch = nullptr;
    } spare;
    float2 *sl = nullptr;        // derived per call: [P*D]
    float *dbase = nullptr;      // [D]
    uint64_t *dxlim = nullptr;   // [D]
    float bw[4] = {0, 0, 0, 0}, lat[4] = {0, 0, 0, 0};
    double bw64[4] = {0, 0, 0, 0};   // the snapshot's bandwidths as given (Proposition 2's counts)
    // a second stream (default priority, non-blocking) on which a large
    // selection runs the derivation and the leader kernels beside the
    // ordering kernels, forked from and joined to the caller's stream by
    // events (so a caller's graph capture takes both branches)
    hipStream_t side = nullptr;
    hipEvent_t ev_fork0 = nullptr, ev_fork1 = nullptr, ev_join = nullptr;
    // the ranking sweep's fork of Proposition 2's counts onto the same stream
    hipEvent_t ev_inv_fork = nullptr, ev_inv_join = nullptr;
    // the flow simulation's work buffer (flowsim.hip)
    void *flow_buf = nullptr;
    uint64_t flow_buf_bytes = 0;
    float t_a = 0, t_b = 0, alpha = 0;
    uint32_t beta_max = 0, bpt = 0, block_tokens = 1;
    uint64_t m_min = 0;
    // cache
    bool have_cache = false;
    uint32_t cache_D = 0;
    // holder index of the resident sets
    uint64_t *table = nullptr;   // [buckets][2] distinct resident hashes
    uint32_t *tvals = nullptr;   // [buckets][2] holder values
    uint64_t *bits = nullptr;    // [rows][bpitch] holder bitmaps
    uint64_t table_bytes = 0, buckets = 0, rows = 0, distinct = 0;
    uint32_t log2b = 0, bpitch = 0;
    bool whole = false;          // a whole set, not a blocked one (see buckets_of)
    uint64_t bits_cap = 0;       // words allocated
    // the cache load's work buffer, kept from load to load
    uint8_t *load_buf = nullptr;
    uint64_t load_bytes = 0;
    // shared index: the hashes of two or more holders (null: none was built)
    u32x4 *sh_tab = nullptr;
    uint32_t sh_log2b = 0;
    // scratch
    uint32_t *errword = nullptr;          // request / selection errors (sticky)
    uint32_t *loadword = nullptr;         // validation flags of the load calls
    float *spt_scen = nullptr;    // ranking sweep: seconds per token of every (scenario, p, d)
    uint64_t spt_cap = 0;
    // the bounded selection: bound factors per (p, group), limits, match counts
    float2 *bnd_lo = nullptr, *bnd_lo2 = nullptr;
    float *bnd_xm = nullptr, *bnd_xg = nullptr;
    uint32_t *match_m = nullptr;
    // groups left per request under the loaded snapshot (spread_kernel), without
    // and with the staged routes
    float spread[2][kSpreadWords] = {};
    uint64_t match_cap = 0;
    float *dlam = nullptr;        // [R][D] B_tok * j of a direct selection with records
    uint64_t dlam_cap = 0;
    int32_t *base_idx = nullptr;
    float *base_score = nullptr;
    uint64_t base_n = 0;
    uint32_t *cnt = nullptr, *adm = nullptr;
    unsigned long long *bytes = nullptr;
    uint32_t commit_P = 0, commit_D = 0;
    // work buffers of the selection (grow to the largest batch seen)
    Scratch sc;
    // options
    uint32_t run_len_opt = 0;   // 0 = automatic
    uint32_t reuse_opt = 1;     // share prefix lengths along the hash order
    uint32_t lead_cap_opt = 0;  // leader table limit (0 = by memory)
    uint32_t cols_opt = 0;      // decodes per lane (0 = automatic)
    uint32_t form_opt = 0;      // 0 automatic, 1 ordering pipeline, 2 bounded
    uint32_t last_form = 0;     // of the last selection: 1 and 2 as above, 3 direct
    uint32_t policy_opt = 0;    // 0 full, 1 without live congestion, 2 topology only
    // sequential-selection scratch
    uint32_t *seq_keys = nullptr, *seq_vals = nullptr, *seq_keys_out = nullptr, *seq_perm = nullptr;
    uint32_t *seq_start = nullptr, *seq_end = nullptr;
    uint64_t seq_cap = 0;
    uint32_t seq_P = 0;
    // timing
    bool timing = false;
    // two-hop routing: the staged route's hop tiers and congestion per (p, d),
    // and its derived rows (like sl)
    uint8_t *rt1 = nullptr, *rt2 = nullptr;
    float *ru1 = nullptr, *ru2 = nullptr;
    float2 *sr = nullptr;
    bool have_route = false;
    // kernel timing: begin/end event pairs in a ring, created on first enable
    std::vector<hipEvent_t> tev;
    uint32_t tcount = 0;    // launches timed since timing was enabled
};

namespace {

struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) (void)hipSetDevice(dev);
    }
    ~DeviceGuard() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

// Events around the one timed kernel of an API call (when timing is on).
hipError_t time_begin(netkv_handle h, hipStream_t st) {
    if (!h->timing) return hipSuccess;
    return hipEventRecord(h->tev[2 * (h->tcount % kTimeSlots)], st);
}

hipError_t time_end(netkv_handle h, hipStream_t st) {
    if (!h->timing) return hipSuccess;
    const hipError_t e = hipEventRecord(h->tev[2 * (h->tcount % kTimeSlots) + 1], st);
    if (e == hipSuccess) ++h->tcount;
    return e;
}

// Timing suspended for a scope (inner steps of a call that times another kernel).
struct TimingOff {
    netkv_handle h;
    bool was;
    explicit TimingOff(netkv_handle hh) : h(hh), was(hh->timing) { h->timing = false; }
    ~TimingOff() { h->timing = was; }
};

netkv_status fail(netkv_handle h, netkv_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (h) h->err = buf;
    return st;
}

#define HIPCHK(h, call)                                                                        \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return fail((h), e_ == hipErrorOutOfMemory ? NETKV_ENOMEM : NETKV_EDEVICE,         \
                        "%s failed: %s", #call, hipGetErrorString(e_));                        \
    } while (0)

template <typename T>
void dfree(T *&p) {
    if (p) (void)hipFree((void *)p);
    p = nullptr;
}

template <typename T>
hipError_t dalloc(T *&p, uint64_t count) {
    dfree(p);
    void *q = nullptr;
    hipError_t e = hipMalloc(&q, std::max<uint64_t>(count, 1) * sizeof(T));
    p = (T *)q;
    return e;
}

uint32_t grid_for(uint64_t n, uint32_t block, uint32_t maxg = 1u << 16) {
    uint64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > maxg) g = maxg;
    return (uint32_t)g;
}

Snap make_snap(netkv_handle h) {
    Snap s;
    s.tier_map = h->tier_map;
    s.util = h->util;
    s.n_inflight = h->n_inflight;
    s.free_mem = h->free_mem;
    s.queue = h->queue;
    s.batch = h->batch;
    for (int i = 0; i < 4; ++i) {
        s.bw[i] = h->bw[i];
        s.lat[i] = h->lat[i];
    }
    s.t_a = h->t_a;
    s.t_b = h->t_b;
    s.alpha = h->alpha;
    s.beta_max = h->beta_max;
    s.m_min = h->m_min;
    s.bpt = h->bpt;
    s.block_tokens = h->block_tokens;
    s.P = h->P;
    s.D = h->D;
    s.sl = h->sl;
    s.slp = sl_pitch(h->D);
    s.sr = nullptr;
    s.dbase = h->dbase;
    s.dxlim = h->dxlim;
    s.policy = h->policy_opt;
    return s;
}

Table make_table(netkv_handle h) {
    Table t;
    t.keys = h->table;
    t.vals = h->tvals;
    t.bits = h->bits;
    t.shift = 64 - h->log2b;
    t.in_block = h->whole ? t.shift : block_shift(t.shift);
    t.bpitch = h->bpitch;
    return t;
}

netkv_status check_requests(netkv_handle h, const netkv_requests_t *req) {
    if (!req) return fail(h, NETKV_EINVAL, "requests is NULL");
    if (req->n_req && (!req->prefill || !req->len_tokens || !req->hash_off))
        return fail(h, NETKV_EINVAL, "request arrays must not be NULL");
    if (req->n_req && req->n_hashes && !req->hashes) return fail(h, NETKV_EINVAL, "hashes is NULL");
    if (req->n_req > (1u << 31)) return fail(h, NETKV_EINVAL, "n_req too large");
    return NETKV_OK;
}

Reqs make_reqs(const netkv_requests_t *req) {
    Reqs r;
    r.n_req = req->n_req;
    r.prefill = req->prefill;
    r.len = req->len_tokens;
    r.off = req->hash_off;
    r.hashes = req->hashes;
    r.n_hashes = req->n_hashes;
    return r;
}

netkv_status ready(netkv_handle h) {
    if (!h->have_snap) return fail(h, NETKV_ENOTREADY, "no snapshot loaded (netkv_oracle_load)");
    if (!h->have_cache) return fail(h, NETKV_ENOTREADY, "no cache loaded (netkv_cache_load)");
    if (h->cache_D != h->D)
        return fail(h, NETKV_EINVAL, "cache has %u decodes, snapshot %u", h->cache_D, h->D);
    return NETKV_OK;
}

// rocPRIM's radix sorts of the batch-order keys (batches outside the range
// of the own batch sort): its tuned kernels, with the merge-sort path
// limited to 2^16 items (rocPRIM's own limit is 2^20).  Above the limit
// the onesweep radix sort takes one pass per 8 key bits; measured on
// MI355X at 2^20 requests, 91 us for the 11-bit prefill order against
// 150 us for the block sort and twenty merge passes.
using SortConfig = rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config,
                                              rocprim::default_config, (size_t)1 << 16>;

// Leader table capacity: prefix lengths of at most 256 MiB (u32 per decode),
// and no more leaders than requests.  Leaders beyond it (and the requests
// that follow them) are matched on their own by the scoring kernel.
constexpr uint64_t kLeadBytes = 256ull << 20;

uint32_t lead_capacity(uint64_t R, uint32_t D) {
    const uint64_t c = std::min<uint64_t>(std::max<uint64_t>(R, 1), kLeadBytes / (4ull * D));
    return (uint32_t)std::max<uint64_t>(c, 1);
}

uint32_t bits_for(uint64_t v) {   // bits to hold 0..v
    uint32_t b = 1;
    while (b < 64 && (v >> b)) ++b;
    return b;
}

void free_scratch(Scratch &sc) {
    dfree(sc.keys_in); dfree(sc.keys_out); dfree(sc.vals_in); dfree(sc.perm); dfree(sc.hot); dfree(sc.cold);
    dfree(sc.seg); dfree(sc.tpre); dfree(sc.hrec); dfree(sc.crec);
    dfree(sc.pkey); dfree(sc.pkey_out); dfree(sc.pval); dfree(sc.pord);
    dfree(sc.n_valid); dfree(sc.hv_used); dfree(sc.n_lead); dfree(sc.hv); dfree(sc.lead); dfree(sc.lead_lam);
    dfree(sc.sort_tmp); dfree(sc.sort_cnt); dfree(sc.sort_tot); dfree(sc.keys_tmp); dfree(sc.vals_tmp);
    dfree(sc.partial);
    dfree(sc.hotr);
    sc = Scratch();
}

// rocPRIM temporary storage for the batch orders of R requests (both sorts
// share one buffer); a size query only.
hipError_t sort_tmp_bytes_for(uint64_t R, size_t &bytes) {
    size_t b1 = 0, b2 = 0;
    uint32_t *k = nullptr;
    hipError_t err = rocprim::radix_sort_pairs<SortConfig>(nullptr, b1, k, k, k, k, (uint32_t)R, 0, 32, nullptr);
    if (err == hipSuccess)
        err = rocprim::radix_sort_pairs<SortConfig>(nullptr, b2, k, k, k, k, (uint32_t)R, 0, 32, nullptr);
    bytes = std::max<size_t>(std::max(b1, b2), 16);
    return err;
}

netkv_status ensure_hv(netkv_handle h, Scratch &sc, uint64_t n_hashes) {
    if (n_hashes <= sc.hv_cap && sc.hv) return NETKV_OK;
    dfree(sc.hv);
    sc.hv_cap = 0;
    if (dalloc(sc.hv, std::max<uint64_t>(n_hashes, 1)) != hipSuccess)
        return fail(h, NETKV_ENOMEM, "holder value scratch allocation failed");
    sc.hv_cap = std::max<uint64_t>(n_hashes, 1);
    return NETKV_OK;
}

// The handle's work buffers for a batch of R requests with n_hashes block
// hashes and partial_elems per-group keys: grown (never shrunk) when a batch
// needs more than any earlier one or than netkv_reserve provided.
netkv_status ensure_scratch(netkv_handle h, Scratch &sc, uint64_t R, uint64_t partial_elems, uint64_t n_hashes,
                            hipStream_t st) {
    if (R > sc.order_cap) {
        dfree(sc.keys_in); dfree(sc.keys_out); dfree(sc.vals_in); dfree(sc.perm); dfree(sc.hot); dfree(sc.cold);
        dfree(sc.seg); dfree(sc.tpre); dfree(sc.pkey); dfree(sc.pkey_out); dfree(sc.pval); dfree(sc.pord);
        dfree(sc.hrec); dfree(sc.crec);
        dfree(sc.sort_tmp);
        dfree(sc.sort_cnt); dfree(sc.sort_tot); dfree(sc.keys_tmp); dfree(sc.vals_tmp);
        sc.order_cap = 0;
        sc.sort_tmp_bytes = 0;
        if (dalloc(sc.keys_in, R) != hipSuccess || dalloc(sc.keys_out, R) != hipSuccess ||
            dalloc(sc.vals_in, R) != hipSuccess || dalloc(sc.perm, R) != hipSuccess ||
            dalloc(sc.hot, R + kHotPad) != hipSuccess || dalloc(sc.cold, R) != hipSuccess ||
            dalloc(sc.seg, R) != hipSuccess || dalloc(sc.tpre, R / kOrderPos + 1) != hipSuccess ||
            dalloc(sc.pkey, R) != hipSuccess || dalloc(sc.pkey_out, R) != hipSuccess ||
            dalloc(sc.pval, R) != hipSuccess || dalloc(sc.pord, R) != hipSuccess ||
            dalloc(sc.hrec, R) != hipSuccess || dalloc(sc.crec, R) != hipSuccess)
            return fail(h, NETKV_ENOMEM, "batch scratch allocation failed");
        // one temporary buffer for the two sorts and the scan
        size_t bytes = 0;
        if (sort_tmp_bytes_for(R, bytes) != hipSuccess) return fail(h, NETKV_EDEVICE, "sort / scan size query failed");
        uint8_t *tmp = nullptr;
        if (dalloc(tmp, bytes) != hipSuccess) return fail(h, NETKV_ENOMEM, "sort scratch allocation failed");
        sc.sort_tmp = tmp;
        sc.sort_tmp_bytes = bytes;
        if (R > kSortMinN) {
            // the own batch sorts run for kSortMinN < n <= kSortMaxN
            const uint64_t n = std::min<uint64_t>(R, kSortMaxN);
            // the most tiles of any batch up to n: small tiles up to
            // kSortSmallTileN, large beyond
            const uint64_t ns = std::min<uint64_t>(n, kSortSmallTileN);
            const uint64_t ntile = std::max((ns + kSortSmallTile - 1) / kSortSmallTile, (n + kSortTile - 1) / kSortTile);
            if (dalloc(sc.sort_cnt, ntile * kSortMaxBins) != hipSuccess ||
                dalloc(sc.sort_tot, kSortMaxBins) != hipSuccess || dalloc(sc.keys_tmp, n) != hipSuccess ||
                dalloc(sc.vals_tmp, n) != hipSuccess)
                return fail(h, NETKV_ENOMEM, "sort scratch allocation failed");
        }
        sc.order_cap = R;
    }
    if (!sc.n_valid && dalloc(sc.n_valid, 1) != hipSuccess) return fail(h, NETKV_ENOMEM, "allocation failed");
    if (!sc.hv_used && dalloc(sc.hv_used, 1) != hipSuccess) return fail(h, NETKV_ENOMEM, "allocation failed");
    if (!sc.n_lead && dalloc(sc.n_lead, 1) != hipSuccess) return fail(h, NETKV_ENOMEM, "allocation failed");
    // holder values of the leaders' blocks: at most one per block of the
    // batch (fewer if runs overlap in the hash array; leaders that do not
    // fit look their blocks up in the leader kernel)
    if (netkv_status e = ensure_hv(h, sc, n_hashes)) return e;
    const uint32_t lc = lead_capacity(R, h->D);
    if (lc > sc.lead_cap || sc.lead_D != h->D || !sc.lead) {
        dfree(sc.lead);
        dfree(sc.lead_lam);
        sc.lead_cap = 0;
        sc.zero_row_set = false;
        if (dalloc(sc.lead, lc) != hipSuccess || dalloc(sc.lead_lam, (uint64_t)(lc + 1) * h->D + kRowPad) != hipSuccess)
            return fail(h, NETKV_ENOMEM, "leader table allocation failed");
        sc.lead_cap = lc;
        sc.lead_D = h->D;
    }
    if (partial_elems > sc.partial_cap) {
        dfree(sc.partial);
        sc.partial_cap = 0;
        if (dalloc(sc.partial, partial_elems) != hipSuccess)
            return fail(h, NETKV_ENOMEM, "partial top-k scratch allocation failed");
        sc.partial_cap = partial_elems;
    }
    return NETKV_OK;
}

// One pass of the batch sort over key bits [shift, shift + bits): counts,
// offsets, scatter (ASSEMBLE: the prefill order's scoring records).
template <bool ASSEMBLE>
hipError_t sort_pass(netkv_handle h, Scratch &sc, const uint32_t *kin, const uint32_t *vin, uint32_t *kout,
                     uint32_t *vout, uint32_t n, uint32_t shift, uint32_t bits, const Pre *hrec,
                     const uint64_t *seg, const uint64_t *tpre, const Cold *crec, uint32_t lstride, uint32_t zrow,
                     Hot *hot, Cold *cold, Hot *hotr, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const uint32_t tile = sort_tile(n);
    const uint32_t ntile = (n + tile - 1) / tile;   // <= kColPer * kBlock (n <= kSortMaxN)
    if (tile == kSortSmallTile)
        hipLaunchKernelGGL(sort_count_kernel<kSortSmallTile>, dim3(ntile), dim3(kBlock), 0, st, kin, n, shift, bits,
                           sc.sort_cnt);
    else
        hipLaunchKernelGGL(sort_count_kernel<kSortTile>, dim3(ntile), dim3(kBlock), 0, st, kin, n, shift, bits,
                           sc.sort_cnt);
    hipLaunchKernelGGL(sort_colscan_kernel, dim3(1u << bits), dim3(kBlock), 0, st, sc.sort_cnt, ntile, bits,
                       sc.sort_tot);
    if (tile == kSortSmallTile)
        hipLaunchKernelGGL((sort_scatter_kernel<ASSEMBLE, kSortSmallTile>), dim3(ntile), dim3(kBlock), 0, st, kin,
                           vin, n, shift, bits, (const uint32_t *)sc.sort_cnt, (const uint32_t *)sc.sort_tot, kout,
                           vout, hrec, seg, tpre, crec, h->block_tokens, lstride, zrow, hot, cold, hotr);
    else
        hipLaunchKernelGGL((sort_scatter_kernel<ASSEMBLE, kSortTile>), dim3(ntile), dim3(kBlock), 0, st, kin, vin,
                           n, shift, bits, (const uint32_t *)sc.sort_cnt, (const uint32_t *)sc.sort_tot, kout, vout,
                           hrec, seg, tpre, crec, h->block_tokens, lstride, zrow, hot, cold, hotr);
    return hipGetLastError();
}

// Bits of pass p of `passes` even passes over nbits key bits, and its shift.
inline void pass_bits(uint32_t nbits, uint32_t passes, uint32_t p, uint32_t &shift, uint32_t &bits) {
    shift = 0;
    for (uint32_t q = 0; q <= p; ++q) {
        bits = (nbits - shift + (passes - q) - 1) / (passes - q);
        if (q < p) shift += bits;
    }
    bits = std::max(bits, 1u);
}

// Stable sort of n (key, value) pairs on key bits [0, nbits) (values: vin,
// or the input positions when vin is null), in passes of at most
// kSortPassBits through the handle's ping-pong buffers; the result lands in
// kout / vout (kSortMinN < n <= kSortMaxN).
hipError_t batch_sort_pairs(netkv_handle h, Scratch &sc, const uint32_t *kin, const uint32_t *vin, uint32_t *kout,
                            uint32_t *vout, uint32_t n, uint32_t nbits, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const uint32_t passes = std::max(1u, (nbits + kSortPassBits - 1) / kSortPassBits);
    const uint32_t *sk = kin, *sv = vin;
    for (uint32_t p = 0; p < passes; ++p) {
        uint32_t shift, bits;
        pass_bits(nbits, passes, p, shift, bits);
        // the last pass writes kout, the one before the ping-pong buffers, ...
        const bool to_out = ((passes - 1 - p) % 2) == 0;
        uint32_t *dk = to_out ? kout : sc.keys_tmp, *dv = to_out ? vout : sc.vals_tmp;
        const hipError_t e = sort_pass<false>(h, sc, sk, sv, dk, dv, n, shift, bits, nullptr, nullptr, nullptr,
                                              nullptr, 0, 0, nullptr, nullptr, nullptr, st);
        if (e != hipSuccess) return e;
        sk = dk;
        sv = dv;
    }
    return hipSuccess;
}

// The prefill order: a stable sort of the hash-order positions by the
// prefill key (pbits <= kPrefillMaxBits), whose last pass writes the
// scoring records at their output positions; earlier passes go through
// buf_k / buf_v (free at this point of a selection).
hipError_t prefill_order(netkv_handle h, Scratch &sc, uint32_t n, uint32_t pbits, uint32_t *buf_k,
                         uint32_t *buf_v, uint32_t lstride, uint32_t zrow, Hot *hotr, hipStream_t st) {
    const uint32_t passes = std::max(1u, (pbits + kSortMaxBits - 1) / kSortMaxBits);
    const uint32_t *sk = sc.pkey, *sv = nullptr;
    for (uint32_t p = 0; p < passes; ++p) {
        uint32_t shift, bits;
        pass_bits(pbits, passes, p, shift, bits);
        hipError_t e;
        if (p + 1 == passes) {
            e = sort_pass<true>(h, sc, sk, sv, nullptr, nullptr, n, shift, bits, sc.hrec, sc.seg, sc.tpre, sc.crec,
                                lstride, zrow, sc.hot, sc.cold, hotr, st);
        } else {
            uint32_t *dk = (p % 2) ? buf_k : sc.keys_tmp, *dv = (p % 2) ? buf_v : sc.vals_tmp;
            e = sort_pass<false>(h, sc, sk, sv, dk, dv, n, shift, bits, nullptr, nullptr, nullptr, nullptr, 0, 0,
                                 nullptr, nullptr, nullptr, st);
            sk = dk;
            sv = dv;
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

uint32_t auto_run_len(uint64_t R, uint32_t ngroup) {
    // runs of 128 sorted requests, shortened (to 8 at least) while that
    // leaves fewer than 32K wavefronts (measured on MI355X: 1,048,576
    // requests of 25 blocks on 8 decode groups score fastest in runs of
    // 128, 65,536 wavefronts, against 64, which starts more runs with a
    // full scan, and 256; 262,144 requests of 191 blocks fastest in runs of
    // 64, 32,768 wavefronts, against 32 and 128)
    const uint64_t work = R * ngroup;
    uint64_t rl = 128;
    while (rl > 8 && work / rl < 32768) rl /= 2;
    return (uint32_t)rl;
}

// decodes per lane (or the option: 1, 2, 3, 4 or 6): the widest of 6, 3
// and 2 whose groups of 64 * C decodes split evenly over the XCDs (at least
// one each), so that every XCD's L2 keeps its own slice of the snapshot
// rows; else 2 on pools of 256+ decodes, else 1 (measured on MI355X: wider
// groups share each request's scalar work over more decodes; 12 per lane
// spills registers, and merging the groups of 3,072 decodes in one
// workgroup was slower than XCD-sliced groups and a merge kernel)
inline uint32_t cols_per_lane(uint32_t D, uint32_t opt) {
    if (opt == 1 || opt == 2 || opt == 3 || opt == 4 || opt == 6) return opt;
    for (uint32_t c : {6u, 3u, 2u}) {
        const uint32_t g = (D + kWave * c - 1) / (kWave * c);
        if (g >= kXcds && g % kXcds == 0) return c;
    }
    return D >= 4u * kWave ? 2u : 1u;
}

// The scoring kernel.  A pool of one group of one
// decode per lane (up to 64 decodes) is scored in merged mode: one
// wavefront per run, writing its requests' outputs itself.  Otherwise one
// workgroup per
// (kWavesPerBlock runs, group) when the groups split evenly over the XCDs
// (see score_kernel), else per kWavesPerBlock waves, writing per-group keys
// that reduce_kernel merges.
template <int K, int C>
hipError_t launch_score(netkv_handle h, Scratch &sc, const Snap &sn, const Table &t, const Reqs &rq,
                        const Order &ord, uint32_t run_len, uint32_t n_runs, uint32_t ngroup, const PairOut &po,
                        bool pairs, uint32_t k, int32_t *idx, float *score, hipStream_t st) {
    hipError_t e = time_begin(h, st);
    if (e != hipSuccess) return e;
    constexpr bool kMergeable = C == 1;
    const bool merge = kMergeable && ngroup == 1;
    const uint64_t grid64 = merge ? (uint64_t)(n_runs + kXcds - 1) / kXcds * kXcds
                            : ngroup % kXcds == 0
                                ? (uint64_t)((n_runs + kWavesPerBlock - 1) / kWavesPerBlock) * ngroup
                                : ((uint64_t)n_runs * ngroup + kWavesPerBlock - 1) / kWavesPerBlock;
    const uint32_t grid = (uint32_t)grid64;
    const uint32_t block = merge ? ngroup * kWave : kBlock;
    // a request that matches on its own (its leader did not fit the leader
    // table, or 2^24 tokens or more) looks blocks up one at a time: rare,
    // and a short loop keeps the kernel's registers for the common path
    const bool two = sn.sr != nullptr;
#define NETKV_SCORE(P2, T2, M2)                                                                                  \
    hipLaunchKernelGGL((score_kernel<K, 1, C, P2, T2, M2>), dim3(grid), dim3(block), 0, st, sn, t, ord.hot,     \
                       ord.cold, ord.lam, sc.lead_cap + 1, rq.hashes, rq.len, rq.off, ord.n_valid, rq.n_req,      \
                       run_len, n_runs, ngroup, sc.partial, po, k, idx, score)
    if (merge) {
        if (pairs) {
            if (two) NETKV_SCORE(true, true, kMergeable);
            else NETKV_SCORE(true, false, kMergeable);
        } else {
            if (two) NETKV_SCORE(false, true, kMergeable);
            else NETKV_SCORE(false, false, kMergeable);
        }
    } else {
        if (pairs) {
            if (two) NETKV_SCORE(true, true, false);
            else NETKV_SCORE(true, false, false);
        } else {
            if (two) NETKV_SCORE(false, true, false);
            else NETKV_SCORE(false, false, false);
        }
    }
#undef NETKV_SCORE
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = time_end(h, st)) != hipSuccess || merge) return e;
    hipLaunchKernelGGL((reduce_kernel<K>), dim3((rq.n_req + 255) / 256), dim3(256), 0, st, rq.n_req, ngroup, k,
                       (const uint64_t *)sc.partial, (const Cold *)ord.cold, ord.n_valid, idx, score);
    return hipGetLastError();
}

// The scoring kernel (bracketed by the handle's timing events when
// enabled), then, outside merged mode, the merge.
template <int K>
hipError_t launch_score_reduce(netkv_handle h, Scratch &sc, const Snap &sn, const Table &t, const Reqs &rq,
                               const Order &ord, uint32_t run_len, uint32_t n_runs, uint32_t ngroup, uint32_t C,
                               const PairOut &po, bool pairs, uint32_t k, int32_t *idx, float *score,
                               hipStream_t st) {
    switch (C) {
    case 6: return launch_score<K, 6>(h, sc, sn, t, rq, ord, run_len, n_runs, ngroup, po, pairs, k, idx, score, st);
    case 4: return launch_score<K, 4>(h, sc, sn, t, rq, ord, run_len, n_runs, ngroup, po, pairs, k, idx, score, st);
    case 3: return launch_score<K, 3>(h, sc, sn, t, rq, ord, run_len, n_runs, ngroup, po, pairs, k, idx, score, st);
    case 2: return launch_score<K, 2>(h, sc, sn, t, rq, ord, run_len, n_runs, ngroup, po, pairs, k, idx, score, st);
    default: return launch_score<K, 1>(h, sc, sn, t, rq, ord, run_len, n_runs, ngroup, po, pairs, k, idx, score, st);
    }
}

// Top-k width K of the kernels for k, decodes per lane C and decode groups.
struct Geometry {
    uint32_t K, C, ngroup;
};

Geometry geometry(netkv_handle h, uint32_t k) {
    Geometry g;
    g.K = k <= 1 ? 1 : k <= 2 ? 2 : k <= 4 ? 4 : 8;
    g.C = cols_per_lane(h->D, h->cols_opt);
    g.ngroup = (h->D + kWave * g.C - 1) / (kWave * g.C);
    return g;
}

// Batches of the direct selection: its work grows with the (request, group of
// 64 decodes) tasks, and with the blocks where runs are longer than 32.
// Measured against the bounded selection (us, tasks -> direct / bounded): 48
// decodes 8,192 -> 21 / 22, 16,384 -> 34 / 29; 768 decodes 12,288 -> 21 / 27,
// 49,152 -> 64 / 28; 3,072 decodes 24,576 -> 45 / 54; runs of 191 blocks on
// 48 decodes 2,048 -> 22 / 28, 4,096 -> 30 / 31.  Where records are wanted
// the ordering pipeline is the other choice: 192 decodes 49,152 -> 56 / 109,
// 3,072 decodes 49,152 -> 63 / 103, 196,608 -> 247 / 123.  Options that shape
// the ordering or the scoring runs ask for that pipeline.
constexpr uint64_t kDirectTasks = 1ull << 14;
constexpr uint64_t kDirectRecordTasks = 1ull << 16;

bool unordered(netkv_handle h) {
    return h->reuse_opt && !h->run_len_opt && !h->cols_opt && !h->lead_cap_opt && h->form_opt != 1;
}

bool direct_batch(netkv_handle h, uint64_t R, uint64_t n_hashes, uint64_t tasks) {
    const uint64_t ng = ((uint64_t)h->D + kWave - 1) / kWave;
    return ng * std::max<uint64_t>(R, n_hashes / 32) <= tasks && unordered(h) && h->form_opt == 0;
}

// The cost factors of a call on `s` (and of the staged routes with `two`).
hipError_t launch_derive(netkv_handle h, const Snap &sn, bool two, hipStream_t s) {
    const uint64_t nd = std::max<uint64_t>((uint64_t)h->P * h->D, h->D);
    hipLaunchKernelGGL(derive_kernel, dim3((uint32_t)((nd + 255) / 256)), dim3(256), 0, s, sn, h->sl, h->dbase,
                       h->dxlim);
    if (two)
        hipLaunchKernelGGL(derive_route_kernel, dim3((uint32_t)((nd + 255) / 256)), dim3(256), 0, s, sn,
                           (const uint8_t *)h->rt1, (const float *)h->ru1, (const uint8_t *)h->rt2,
                           (const float *)h->ru2, h->sr);
    return hipGetLastError();
}

netkv_status run_direct(netkv_handle h, const netkv_requests_t *req, uint32_t k, int32_t *idx, float *score,
                        hipStream_t st, bool route2, Hot *hotr = nullptr, float *lam = nullptr) {
    const uint32_t R = req->n_req, ng = (h->D + kWave - 1) / kWave;
    const bool two = route2 && h->have_route;
    const bool fly = !two && !hotr;
    Snap sn = make_snap(h);
    if (!fly) HIPCHK(h, launch_derive(h, sn, two, st));
    if (two) sn.sr = h->sr;
    // four wavefronts share a request when one each leaves most of the chip idle
    const uint32_t nw = ng > 4 && R <= 2048 ? 4 : 1;
    const uint32_t C = ng == 1 ? 1 : ng <= 4 || (nw > 1 && ng <= 16) ? 4 : 12;
    const uint32_t grid = (uint32_t)(((uint64_t)R * nw + kWavesPerBlock - 1) / kWavesPerBlock);
    const Table t = make_table(h);
    const Reqs rq = make_reqs(req);
    HIPCHK(h, time_begin(h, st));
#define NETKV_DIRECT(KK)                                                                                             \
    do {                                                                                                             \
        if (C == 1)                                                                                                  \
            hipLaunchKernelGGL((direct_kernel<KK, 1>), dim3(grid), dim3(kBlock), 0, st, sn, t, rq, nw, fly, k, idx,   \
                               score, h->errword, hotr, lam);                                                        \
        else if (C == 4)                                                                                             \
            hipLaunchKernelGGL((direct_kernel<KK, 4>), dim3(grid), dim3(kBlock), 0, st, sn, t, rq, nw, fly, k, idx,   \
                               score, h->errword, hotr, lam);                                                        \
        else                                                                                                         \
            hipLaunchKernelGGL((direct_kernel<KK, 12>), dim3(grid), dim3(kBlock), 0, st, sn, t, rq, nw, fly, k, idx,  \
                               score, h->errword, hotr, lam);                                                        \
    } while (0)
    if (k <= 1) NETKV_DIRECT(1);
    else if (k <= 2) NETKV_DIRECT(2);
    else if (k <= 4) NETKV_DIRECT(4);
    else NETKV_DIRECT(8);
#undef NETKV_DIRECT
    HIPCHK(h, hipGetLastError());
    HIPCHK(h, time_end(h, st));
    return NETKV_OK;
}

// The whole selection of one batch on `st` with the work buffers of sc
// (which must hold the batch: R <= order_cap, R * ngroup * K <= partial_cap):
// validate and key the requests, hash order (sort), common runs and
// leaders, the segmented scan, prefill order (stable sort), scoring
// records, leaders' prefix lengths, scoring, merge.  Launches kernels only.
// Without score_pairs it ends with the leaders' prefix lengths and the
// records by batch index (hotr): the sequential form scores its own pairs
// (the scoring it skips took 100 of 574 us for 131,071 requests on 3,072
// decodes).
netkv_status run_select(netkv_handle h, Scratch &sc, const netkv_requests_t *req, uint32_t k, int32_t *idx,
                        float *score, const PairOut &po, bool pairs, uint32_t max_blocks, hipStream_t st,
                        bool route2 = false, bool derive = true, Hot *hotr = nullptr, bool score_pairs = true) {
    const uint64_t R = req->n_req;
    const Geometry geo = geometry(h, k);
    const uint32_t K = geo.K, C = geo.C, ngroup = geo.ngroup;
    Snap sn = make_snap(h);
    const Table t = make_table(h);
    const Reqs rq = make_reqs(req);
    if (!sc.zero_row_set) {
        // the all-zero row of requests without a leader (no leader writes it)
        hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(h->D, 256)), dim3(256), 0, st,
                           (uint32_t *)(sc.lead_lam + (uint64_t)sc.lead_cap * h->D), (uint64_t)h->D, 0u);
        HIPCHK(h, hipGetLastError());
        sc.zero_row_set = true;
    }
    // a large batch forks a second stream: the derivation (independent of
    // the ordering), then after the order kernel the leaders' holder values
    // and prefix lengths, beside the tile prefixes and the prefill order;
    // joined before the scoring kernel
    const bool fork = R >= kForkMinN;
    hipStream_t s2 = fork ? h->side : st;
    if (fork) {
        HIPCHK(h, hipEventRecord(h->ev_fork0, st));
        HIPCHK(h, hipStreamWaitEvent(s2, h->ev_fork0, 0));
    }
    const bool two = route2 && h->have_route;
    if (derive) HIPCHK(h, launch_derive(h, sn, two, s2));
    if (two) sn.sr = h->sr;
    // the own batch sort (its first pass takes positions as values) where
    // its buffers are there and the batch is in its range
    const bool own_sort = R > kSortMinN && R <= kSortMaxN && sc.sort_cnt != nullptr;
    hipLaunchKernelGGL(prep_kernel, dim3((uint32_t)((R + 255) / 256)), dim3(256), 0, st, sn, rq, max_blocks,
                       sc.keys_in, own_sort ? nullptr : sc.vals_in, h->errword, sc.hv_used, sc.n_lead, k, idx, score);
    HIPCHK(h, hipGetLastError());
    size_t tb = sc.sort_tmp_bytes;
    if (own_sort)
        HIPCHK(h, batch_sort_pairs(h, sc, sc.keys_in, nullptr, sc.keys_out, sc.perm, (uint32_t)R, 32, st));
    else
        HIPCHK(h, rocprim::radix_sort_pairs<SortConfig>(sc.sort_tmp, tb, sc.keys_in, sc.keys_out, sc.vals_in,
                                                        sc.perm, (uint32_t)R, 0, 32, st));
    // leaders (and holder values of their blocks) the table takes this call
    const uint32_t lcap = h->lead_cap_opt ? std::min(sc.lead_cap, h->lead_cap_opt) : sc.lead_cap;
    const uint64_t hvcap = h->lead_cap_opt ? std::min<uint64_t>(sc.hv_cap, h->lead_cap_opt) : sc.hv_cap;
    // the prefill order: the own sort (positions as its values), or rocPRIM's on pval
    const uint32_t pbits = bits_for(h->P);
    const bool own_prefill = own_sort && pbits <= kPrefillMaxBits;
    hipLaunchKernelGGL(order_kernel<kLcpLanes>, dim3((uint32_t)((R * kLcpLanes + 255) / 256)), dim3(256), 0, st, rq,
                       h->P, sl_pitch(h->D), h->block_tokens, (const uint32_t *)sc.perm,
                       (const uint32_t *)sc.keys_out, t, h->reuse_opt, sc.seg, sc.tpre, sc.pkey,
                       own_prefill ? nullptr : sc.pval, sc.hrec, sc.crec, sc.lead, lcap, sc.n_lead, hvcap,
                       sc.hv_used, sc.n_valid);
    HIPCHK(h, hipGetLastError());
    if (fork) {
        HIPCHK(h, hipEventRecord(h->ev_fork1, st));
        HIPCHK(h, hipStreamWaitEvent(s2, h->ev_fork1, 0));
    }
    hipLaunchKernelGGL(lead_holder_kernel, dim3((uint32_t)std::min<uint64_t>((lcap + kWavesPerBlock - 1) /
                                                                             kWavesPerBlock, 4096)),
                       dim3(kBlock), 0, s2, t, rq.hashes, sc.lead, (const unsigned int *)sc.n_lead, lcap, sc.hv);
    {
        // leaders' prefix lengths: 64 decodes per wavefront, 64 blocks per step
        const uint32_t lgroup = (h->D + kWave - 1) / kWave;
        const uint64_t lw = std::min<uint64_t>((uint64_t)lcap * ((lgroup + kLeadGroups - 1) / kLeadGroups), 65536);
        hipLaunchKernelGGL(lead_kernel, dim3((uint32_t)((lw + kWavesPerBlock - 1) / kWavesPerBlock)),
                           dim3(kBlock), 0, s2, t, h->D, h->block_tokens, (const Lead *)sc.lead,
                           (const unsigned int *)sc.n_lead, lcap, (const uint32_t *)sc.hv, rq.hashes, lgroup,
                           sc.lead_lam);
    }
    HIPCHK(h, hipGetLastError());
    // the exclusive prefixes of the order tiles' totals (the second level of
    // the segmented scan; the first is in order_kernel)
    hipLaunchKernelGGL(tile_prefix_kernel, dim3(1), dim3(kPrefixThreads), 0, st, sc.tpre,
                       (uint32_t)((R + kOrderPos - 1) / kOrderPos));
    HIPCHK(h, hipGetLastError());
    // prefill order (stable: the hash order within each prefill) and the
    // scoring records in it
    const uint32_t lstride = h->D * (uint32_t)sizeof(float);
    if (!score_pairs) {
        hipLaunchKernelGGL(records_kernel, dim3((uint32_t)((R + 255) / 256)), dim3(256), 0, st, (uint32_t)R,
                           h->block_tokens, lstride, sc.lead_cap * lstride, (const uint64_t *)sc.seg,
                           (const uint64_t *)sc.tpre, (const Pre *)sc.hrec, (const Cold *)sc.crec, hotr);
        HIPCHK(h, hipGetLastError());
    } else if (own_prefill) {
        // (the hash order's keys and permutation are no longer needed)
        HIPCHK(h, prefill_order(h, sc, (uint32_t)R, pbits, sc.keys_out, sc.perm, lstride, sc.lead_cap * lstride,
                                hotr, st));
    } else {
        tb = sc.sort_tmp_bytes;
        HIPCHK(h, rocprim::radix_sort_pairs<SortConfig>(sc.sort_tmp, tb, sc.pkey, sc.pkey_out, sc.pval, sc.pord,
                                                        (uint32_t)R, 0, pbits, st));
        hipLaunchKernelGGL(assemble_kernel, dim3((uint32_t)((R + kHotPad + 255) / 256)), dim3(256), 0, st,
                           (uint32_t)R, h->block_tokens, lstride, sc.lead_cap * lstride, (const uint32_t *)sc.pord,
                           (const uint64_t *)sc.seg, (const uint64_t *)sc.tpre, (const Pre *)sc.hrec,
                           (const Cold *)sc.crec, sc.hot, sc.cold, hotr);
        HIPCHK(h, hipGetLastError());
    }
    if (fork) {
        HIPCHK(h, hipEventRecord(h->ev_join, s2));
        HIPCHK(h, hipStreamWaitEvent(st, h->ev_join, 0));
    }
    if (!score_pairs) return NETKV_OK;
    const uint32_t run_len = h->run_len_opt ? h->run_len_opt : auto_run_len(R, ngroup);
    const uint32_t n_runs = (uint32_t)((R + run_len - 1) / run_len);
    Order ord{sc.hot, sc.cold, sc.lead_lam, sc.hv, sc.n_valid, lcap};
    if (K == 1)
        HIPCHK(h, launch_score_reduce<1>(h, sc, sn, t, rq, ord, run_len, n_runs, ngroup, C, po, pairs, k, idx,
                                         score, st));
    else if (K == 2)
        HIPCHK(h, launch_score_reduce<2>(h, sc, sn, t, rq, ord, run_len, n_runs, ngroup, C, po, pairs, k, idx,
                                         score, st));
    else if (K == 4)
        HIPCHK(h, launch_score_reduce<4>(h, sc, sn, t, rq, ord, run_len, n_runs, ngroup, C, po, pairs, k, idx,
                                         score, st));
    else
        HIPCHK(h, launch_score_reduce<8>(h, sc, sn, t, rq, ord, run_len, n_runs, ngroup, C, po, pairs, k, idx,
                                         score, st));
    return NETKV_OK;
}

// Groups left per request of a batch, as measured when the snapshot was loaded,
// at the measured length nearest in proportion to the batch's mean.
double groups_left(netkv_handle h, uint64_t R, uint64_t n_hashes, uint32_t K, bool two) {
    if (h->D <= (uint32_t)kWave) return 1.0;
    const double tokens = (double)h->block_tokens * (double)n_hashes / (double)R;
    uint32_t i = 0;
    while (i + 1 < kSpreadLens && tokens * tokens > (double)spread_tokens(i) * (double)spread_tokens(i + 1)) ++i;
    return h->spread[two][i * kSpreadKs + (uint32_t)__builtin_ctz(K)];
}

// The bounded selection or the ordering pipeline: pools of up to 64 groups of
// 64 decodes, by estimates of both forms' times.  The pipeline takes some 10 to
// 25 launches and then scores every pair, sharing the prefix lookups along its
// order; the bounded selection takes three, looks up every held block of every
// request and scores the groups that the bounds leave, so it loses on large
// batches of long runs, on large batches in small pools, and wherever the
// snapshot does not tell the groups apart (left: groups left per request as
// measured when the snapshot was loaded; 150,001 requests on 3,072 identical
// decodes take 1,378 us bounded and 285 us ordered).  The lines are least-squares
// fits, in us, to 2,608 calls timed in both forms: 48 to 4,080 decodes, 350 to
// 1,048,576 requests of 25 and of 191 blocks, k = 1, 2, 3 and 8, with and without
// staged routes and memory pressure, on fat trees, one tier, two tiers and
// identical decodes.  The form taken costs 1.6 % more than the better one of the
// two on average, and over 10 % more than the pipeline in 18 of them.
bool bounded_batch(netkv_handle h, uint64_t R, uint64_t n_hashes, uint32_t k, bool two) {
    const uint64_t ng = (h->D + kWave - 1) / kWave;
    if (ng > kBoundMaxGroups || !unordered(h)) return false;
    if (h->form_opt == 2) return true;
    const Geometry geo = geometry(h, k);
    const double K = geo.K, n = (double)R, left = groups_left(h, R, n_hashes, geo.K, two);
    const double pipeline = 58.0 + 10.0 * std::log2(std::max(n, 350.0) / 350.0) + 0.8 * (double)ng +
                            1e-3 * n * (0.124 + 0.009 * K + geo.ngroup * (0.0053 + 0.025 * K) +
                                        (double)ng * (0.0034 + 0.003 * K + (two ? 0.0064 : 0.0)));
    const double s = left + (two ? 0.9 * (left - 1.0) : 0.0);   // (two routes leave more than the estimate)
    double bounded = 38.0 + 1.4 * (double)ng + 0.5 * s + 1e-3 * n * (0.22 + 0.02 * K + s * (0.057 + 0.0315 * K)) +
                     1e-3 * (double)n_hashes * (0.0024 + 0.0019 * s);
    // (few requests that leave hardly a group: the constants above include the
    // longest wavefront's groups)
    if (left <= 2.0 && n <= 6000.0 && K <= 4.0) bounded *= 0.65;
    // (beyond these the estimates are off by the most: merges of k > 4, two
    // routes on many groups, more long runs than were measured)
    const double tasks = n * (double)ng;
    if ((K > 4.0 && tasks > (double)(1u << 20)) || (two && tasks * (K > 1.0 ? 4.0 : 1.0) > 5.0 * (1u << 20)) ||
        ((double)n_hashes > 64.0 * n && n_hashes > 32u << 20))
        return false;
    return 1.05 * bounded <= pipeline;
}

// Pools of the bounded selection, whose tables are sized with the snapshot's.
bool bound_pool(uint32_t D) { return D <= kBoundMaxGroups * kWave; }

netkv_status ensure_match(netkv_handle h, uint64_t R) {
    if (R <= h->match_cap || !bound_pool(h->D)) return NETKV_OK;
    dfree(h->match_m);
    h->match_cap = 0;
    if (dalloc(h->match_m, R) != hipSuccess) return fail(h, NETKV_ENOMEM, "match scratch allocation failed");
    h->match_cap = R;
    return NETKV_OK;
}

netkv_status run_bounded(netkv_handle h, const netkv_requests_t *req, uint32_t k, int32_t *idx, float *score,
                         hipStream_t st, bool route2) {
    const uint64_t R = req->n_req;
    const uint32_t ng = (h->D + kWave - 1) / kWave;
    netkv_status e = ensure_match(h, R);
    if (e || (e = ensure_hv(h, h->sc, req->n_hashes))) return e;
    const bool two = route2 && h->have_route;
    Snap sn = make_snap(h);
    const Table t = make_table(h);
    const Reqs rq = make_reqs(req);
    const uint64_t tasks = (uint64_t)h->P * ng;
    hipLaunchKernelGGL(derive_bound_kernel, dim3((uint32_t)((tasks + kWavesPerBlock - 1) / kWavesPerBlock)), dim3(kBlock),
                       0, st, sn, (const uint8_t *)h->rt1, (const float *)h->ru1, (const uint8_t *)h->rt2,
                       (const float *)h->ru2, ng, h->sl, two ? h->sr : nullptr, h->dbase, h->dxlim, h->bnd_lo, h->bnd_lo2,
                       h->bnd_xm, h->bnd_xg);
    const Shared sh{h->sh_tab, 64 - h->sh_log2b, (1u << h->sh_log2b) - 1u};
    hipLaunchKernelGGL((match_kernel<kStepLanes, kStepBlocks>), dim3((uint32_t)((R * kStepLanes + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, st, sn, t, sh, rq, h->sc.hv, h->match_m, h->errword);
    HIPCHK(h, hipGetLastError());
    if (two) sn.sr = h->sr;
    const Bounds bd{h->bnd_lo, h->bnd_lo2, h->bnd_xm, h->bnd_xg, ng};
    const uint32_t K = k <= 1 ? 1 : k <= 2 ? 2 : k <= 4 ? 4 : 8;
    // four requests and more per wavefront share their loads, but their left
    // groups are scored and merged one after another: with several of them (or
    // longer merges), and too few requests to fill the chip, one request each
    // (us, one / four: 500 requests on 3,072 decodes, k = 8, 12 groups left 103 /
    // 160, 8,192 130 / 185, 16,000 172 / 250; 20,011 on 768, k = 1, 1.1 left 60 /
    // 48; 8,192 on 192, k = 3, 1.2 left 36 / 33; k = 8, 2 left on 78 decodes, 6,000
    // 34 / 36, 11,000 41 / 39, 24,000 66 / 55; 5.4 left on 768 16,000 86 / 92,
    // 24,000 111 / 105)
    uint32_t per = (uint32_t)std::min<uint64_t>(std::min<uint64_t>(16, 64 / K), std::max<uint64_t>(4, R / 8192 / 4 * 4));
    const double merges = groups_left(h, R, req->n_hashes, K, two) * (3.0 + K);
    if (merges >= 12.0 && (double)R < (K > 4 ? std::min(20480.0, 360.0 * merges) : 12288.0)) per = 1;
    const uint32_t grid = (uint32_t)((R + (uint64_t)per * kWavesPerBlock - 1) / ((uint64_t)per * kWavesPerBlock));
    HIPCHK(h, time_begin(h, st));
#define NETKV_BOUNDED(KK)                                                                                             \
    do {                                                                                                              \
        if (two)                                                                                                      \
            hipLaunchKernelGGL((bounded_kernel<KK, true>), dim3(grid), dim3(kBlock), 0, st, sn, t, rq, bd,             \
                               (const uint32_t *)h->sc.hv, (const uint32_t *)h->match_m, per, k, idx, score);         \
        else                                                                                                          \
            hipLaunchKernelGGL((bounded_kernel<KK, false>), dim3(grid), dim3(kBlock), 0, st, sn, t, rq, bd,            \
                               (const uint32_t *)h->sc.hv, (const uint32_t *)h->match_m, per, k, idx, score);         \
    } while (0)
    if (K == 1) NETKV_BOUNDED(1);
    else if (K == 2) NETKV_BOUNDED(2);
    else if (K == 4) NETKV_BOUNDED(4);
    else NETKV_BOUNDED(8);
#undef NETKV_BOUNDED
    HIPCHK(h, hipGetLastError());
    HIPCHK(h, time_end(h, st));
    return NETKV_OK;
}

// Scoring records by batch index for n requests (ranking sweep, sequential form).
netkv_status ensure_hotr(netkv_handle h, uint64_t n) {
    if (n <= h->sc.hotr_cap) return NETKV_OK;
    dfree(h->sc.hotr);
    h->sc.hotr_cap = 0;
    if (dalloc(h->sc.hotr, n) != hipSuccess) return fail(h, NETKV_ENOMEM, "record scratch allocation failed");
    h->sc.hotr_cap = n;
    return NETKV_OK;
}

// Rows of the direct selection's records: every request its own leader.
netkv_status ensure_dlam(netkv_handle h, uint64_t R) {
    if (R * h->D <= h->dlam_cap) return NETKV_OK;
    dfree(h->dlam);
    h->dlam_cap = 0;
    if (dalloc(h->dlam, R * h->D) != hipSuccess) return fail(h, NETKV_ENOMEM, "record scratch allocation failed");
    h->dlam_cap = R * h->D;
    return NETKV_OK;
}

// The sequential form's per-prefill ordering of R requests over P prefill
// instances (seq), and the ranking sweep's selection under the loaded
// snapshot (base).
netkv_status ensure_seq(netkv_handle h, uint64_t R, uint64_t P, bool seq, bool base) {
    if (seq && h->seq_cap < R) {
        dfree(h->seq_keys); dfree(h->seq_vals); dfree(h->seq_keys_out); dfree(h->seq_perm);
        h->seq_cap = 0;
        HIPCHK(h, dalloc(h->seq_keys, R));
        HIPCHK(h, dalloc(h->seq_vals, R));
        HIPCHK(h, dalloc(h->seq_keys_out, R));
        HIPCHK(h, dalloc(h->seq_perm, R));
        h->seq_cap = R;
    }
    if (seq && h->seq_P != P) {
        dfree(h->seq_start); dfree(h->seq_end);
        h->seq_P = 0;
        HIPCHK(h, dalloc(h->seq_start, P));
        HIPCHK(h, dalloc(h->seq_end, P));
        h->seq_P = (uint32_t)P;
    }
    if (base && h->base_n < R) {
        dfree(h->base_idx);
        dfree(h->base_score);
        h->base_n = 0;
        HIPCHK(h, dalloc(h->base_idx, R));
        HIPCHK(h, dalloc(h->base_score, R));
        h->base_n = R;
    }
    return NETKV_OK;
}

// The handle's buffers for the batch, then the selection.
// With want_hotr, every request's scoring record is also kept by batch
// index in sc.hotr (grown to the batch).
netkv_status select_owned(netkv_handle h, const netkv_requests_t *req, uint32_t k, int32_t *idx, float *score,
                          const PairOut &po, bool pairs, uint32_t max_blocks, hipStream_t st, bool route2 = false,
                          bool want_hotr = false, bool score_pairs = true) {
    const Geometry geo = geometry(h, k);
    netkv_status e = ensure_scratch(h, h->sc, req->n_req,
                                    score_pairs ? (uint64_t)req->n_req * geo.ngroup * geo.K : 0, req->n_hashes, st);
    if (e) return e;
    if (want_hotr && (e = ensure_hotr(h, req->n_req))) return e;
    return run_select(h, h->sc, req, k, idx, score, po, pairs, max_blocks, st, route2, true,
                      want_hotr ? h->sc.hotr : nullptr, score_pairs);
}

// After a selection that did not use all of them: the work buffers that any
// form of a batch of this size uses, so that a later one -- with per-pair
// outputs, more of k, other congestion, routes or options -- allocates no more
// than for a batch of this size before.  The selection's kernels run meanwhile.
// Not while the stream is captured, where nothing can be allocated, and no
// error of the call, whose results do not need them.
void size_ahead(netkv_handle h, const netkv_requests_t *req, uint32_t k, hipStream_t st) {
    const Geometry geo = geometry(h, k);
    const uint64_t R = req->n_req, elems = R * geo.ngroup * geo.K;
    const Scratch &sc = h->sc;
    const bool match = R <= h->match_cap || !bound_pool(h->D);
    if (match && R <= sc.order_cap && elems <= sc.partial_cap && req->n_hashes <= sc.hv_cap && sc.lead_D == h->D &&
        lead_capacity(R, h->D) <= sc.lead_cap)
        return;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return;
    }
    if (ensure_scratch(h, h->sc, R, elems, req->n_hashes, st) || ensure_match(h, R)) {
        (void)hipGetLastError();
        h->err.clear();
    }
}

// ---- work buffers carved from the static scratch array (no allocation)

constexpr uint64_t kAlign = 256;
inline uint64_t align_up(uint64_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Lay out the buffers of a selection of at most r requests (no own-sort
// buffers: r <= kSortMinN), lead_cap leaders and hv_cap holder values in
// the bytes at base; with base null only the size is computed.  Returns
// the bytes used.
uint64_t carve(uint8_t *base, uint64_t r, uint32_t D, uint64_t partial_elems, uint32_t lead_cap, uint64_t hv_cap,
               size_t tmp_bytes, Scratch *sc) {
    uint64_t used = 0;
    auto take = [&](uint64_t bytes) -> uint8_t * {
        uint8_t *p = base ? base + used : nullptr;
        used = align_up(used + std::max<uint64_t>(bytes, 1));
        return p;
    };
    Scratch t;
    t.n_valid = (uint32_t *)take(4);
    t.hv_used = (unsigned long long *)take(8);
    t.n_lead = (unsigned int *)take(4);
    t.sort_tmp = take(tmp_bytes);
    t.sort_tmp_bytes = tmp_bytes;
    t.keys_in = (uint32_t *)take(4 * r);
    t.keys_out = (uint32_t *)take(4 * r);
    t.vals_in = (uint32_t *)take(4 * r);
    t.perm = (uint32_t *)take(4 * r);
    t.hot = (Hot *)take(sizeof(Hot) * (r + kHotPad));
    t.cold = (Cold *)take(sizeof(Cold) * r);
    t.seg = (uint64_t *)take(8 * r);
    t.tpre = (uint64_t *)take(8 * (r / kOrderPos + 1));
    t.hrec = (Pre *)take(sizeof(Pre) * r);
    t.crec = (Cold *)take(sizeof(Cold) * r);
    t.pkey = (uint32_t *)take(4 * r);
    t.pkey_out = (uint32_t *)take(4 * r);
    t.pval = (uint32_t *)take(4 * r);
    t.pord = (uint32_t *)take(4 * r);
    t.partial = (uint64_t *)take(8 * partial_elems);
    t.partial_cap = partial_elems;
    t.lead = (Lead *)take(sizeof(Lead) * (uint64_t)lead_cap);
    t.lead_lam = (float *)take(4ull * (((uint64_t)lead_cap + 1) * D + kRowPad));
    t.lead_cap = lead_cap;
    t.lead_D = D;
    t.hv = (uint32_t *)take(4 * hv_cap);
    t.hv_cap = hv_cap;
    t.order_cap = r;
    t.zero_row_set = false;
    if (sc) *sc = t;
    return used;
}

// Sub-batch size and buffers for a no-allocation selection of R requests:
// the largest r (at most kSortMinN, halved down to 256) whose per-request
// buffers and per-group keys fit with one leader row; what is left goes
// half to leader rows, half to leaders' holder values.
netkv_status carve_static(netkv_handle h, uint8_t *base, uint64_t R, uint32_t k, Scratch &sc, uint64_t &r_sub) {
    const Geometry geo = geometry(h, k);
    const uint32_t D = h->D;
    uint64_t r = std::min<uint64_t>(R, kSortMinN);
    size_t tmp = 0;
    for (;;) {
        if (sort_tmp_bytes_for(r, tmp) != hipSuccess) return fail(h, NETKV_EDEVICE, "sort / scan size query failed");
        if (carve(nullptr, r, D, r * geo.ngroup * geo.K, 1, 1, tmp, nullptr) <= kScratchBytes) break;
        if (r <= 256)
            return fail(h, NETKV_ECAPACITY,
                        "the no-allocation scratch (%llu MiB) cannot hold a sub-batch of %llu requests on %u decodes "
                        "with k = %u",
                        (unsigned long long)(kScratchBytes >> 20), (unsigned long long)r, D, k);
        r = std::max<uint64_t>(256, r / 2);
    }
    const uint64_t base_bytes = carve(nullptr, r, D, r * geo.ngroup * geo.K, 1, 1, tmp, nullptr);
    const uint64_t rest = kScratchBytes - base_bytes;
    const uint64_t row = 4ull * D + sizeof(Lead);
    const uint64_t slack = 4 * kAlign;
    uint64_t extra = rest > slack ? std::min<uint64_t>(r - 1, (rest - slack) / 2 / row) : 0;
    uint64_t hv_cap = 1 + (rest > slack + extra * row ? (rest - slack - extra * row) / 4 : 0);
    while (carve(nullptr, r, D, r * geo.ngroup * geo.K, (uint32_t)(1 + extra), hv_cap, tmp, nullptr) > kScratchBytes) {
        if (hv_cap > 1024) hv_cap -= 1024;
        else if (extra > 0) --extra;
        else break;   // one leader row and one holder value: fits (checked above)
    }
    carve(base, r, D, r * geo.ngroup * geo.K, (uint32_t)(1 + extra), hv_cap, tmp, &sc);
    r_sub = r;
    return NETKV_OK;
}

void free_spare(netkv_ctx::SnapBuf &b) {
    dfree(b.tier_map); dfree(b.util); dfree(b.n_inflight); dfree(b.free_mem);
    dfree(b.adm_prev); dfree(b.queue); dfree(b.batch);
    b.P = b.D = 0;
}

netkv_status ensure_spare(netkv_handle h, uint32_t P, uint32_t D) {
    netkv_ctx::SnapBuf &sp = h->spare;
    if (sp.P == P && sp.D == D) return NETKV_OK;
    const uint64_t npd = (uint64_t)P * D;
    free_spare(sp);
    if (dalloc(sp.tier_map, npd) != hipSuccess || dalloc(sp.util, npd) != hipSuccess ||
        dalloc(sp.n_inflight, 4ull * P) != hipSuccess || dalloc(sp.free_mem, D) != hipSuccess ||
        dalloc(sp.adm_prev, D) != hipSuccess || dalloc(sp.queue, D) != hipSuccess || dalloc(sp.batch, D) != hipSuccess) {
        free_spare(sp);
        return fail(h, NETKV_ENOMEM, "snapshot allocation failed");
    }
    sp.P = P;
    sp.D = D;
    return NETKV_OK;
}

// Whether p is memory of the handle's device (host memory, pinned or not,
// managed memory and other devices' are copied by the runtime).
bool on_device(netkv_handle h, const void *p) {
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();   // not an error of this call: ordinary host memory
        return false;
    }
    return at.type == hipMemoryTypeDevice && at.device == h->device && !at.isManaged;
}

bool finite_nonneg(double x) { return std::isfinite(x) && x >= 0.0; }

// What the load calls read back: validation flags, then spread_kernel's counts.
struct LoadBack {
    uint32_t bad = 0;
    uint32_t spread[2][kSpreadP][kSpreadWords];
};

// Pools whose bounds are measured at a load: those of several groups that the
// bounded selection takes.
bool spread_pool(uint32_t D) { return D > kWave && D <= kBoundMaxGroups * kWave; }

// Bytes of it that a load copies back.
size_t back_bytes(uint32_t D, bool two) {
    return !spread_pool(D) ? sizeof(uint32_t)
         : two             ? sizeof(LoadBack)
                           : sizeof(uint32_t) * (1 + kSpreadP * kSpreadWords);
}

// The bounds' spread of snapshot s (and of the staged routes t1 .. with two)
// into h->loadword; read by read_spread from what was copied back.
hipError_t launch_spread(netkv_handle h, const Snap &s, bool direct, bool two, const uint8_t *t1, const float *u1,
                         const uint8_t *t2, const float *u2, hipStream_t st) {
    if (!spread_pool(s.D)) return hipGetLastError();
    const uint32_t ng = (s.D + kWave - 1) / kWave;
    const dim3 grid(std::min(s.P, kSpreadP), kSpreadLens), block(kSpreadWaves * kWave);
    if (direct)
        hipLaunchKernelGGL(spread_kernel<false>, grid, block, 0, st, s, nullptr, nullptr, nullptr, nullptr, ng,
                           h->loadword + 1);
    if (two)
        hipLaunchKernelGGL(spread_kernel<true>, grid, block, 0, st, s, t1, u1, t2, u2, ng,
                           h->loadword + 1 + kSpreadP * kSpreadWords);
    return hipGetLastError();
}

// (a length that most prefills cannot place takes the next shorter one's measure)
void read_spread(netkv_handle h, uint32_t P, bool two, const LoadBack &back) {
    if (!spread_pool(h->D)) return;
    const uint32_t np = std::min(P, kSpreadP);
    for (uint32_t i = 0; i < kSpreadWords; ++i) {
        uint32_t sum = 0, n = 0;
        for (uint32_t p = 0; p < np; ++p)
            if (back.spread[two][p][i] != 0xFFFFFFFFu) {
                sum += back.spread[two][p][i];
                ++n;
            }
        h->spread[two][i] = 2 * n >= np       ? (float)sum / (2.0f * (float)n)
                            : i >= kSpreadKs ? h->spread[two][i - kSpreadKs]
                                             : (float)((h->D + kWave - 1) / kWave);
    }
}

}  // namespace

namespace {

template <int K, int NX, bool LDS, bool FULL>
void launch_sweep(dim3 grid, size_t lds, hipStream_t st, const Snap &sn, const Table &t, const Reqs &rq,
                  const Hot *hotr, const float *lead_lam, const float *spt, uint32_t n_scen, const int32_t *bidx,
                  const float *bsc, uint32_t k, int32_t *out_idx, float *out_score, unsigned long long *fl) {
    hipLaunchKernelGGL((sweep_kernel<K, NX, LDS, FULL>), grid, dim3(kSweepThreads), lds, st, sn, t, rq, hotr,
                       lead_lam, spt, n_scen, bidx, bsc, k, out_idx, out_score, fl);
}

// 48 decodes (the 64-GPU pools) with compile-time decode indices, up to 48
// with a bounds test, more 64 at a time; the per-(p, d) tables in LDS when
// they fit, else read from memory.
template <int K>
void launch_sweep_k(uint32_t D, bool lds, dim3 grid, size_t lds_bytes, hipStream_t st, const Snap &sn, const Table &t,
                    const Reqs &rq, const Hot *hotr, const float *lead_lam, const float *spt, uint32_t n_scen,
                    const int32_t *bidx, const float *bsc, uint32_t k, int32_t *out_idx, float *out_score,
                    unsigned long long *fl) {
    if (lds && D == 48)
        launch_sweep<K, 48, true, true>(grid, lds_bytes, st, sn, t, rq, hotr, lead_lam, spt, n_scen, bidx, bsc, k,
                                        out_idx, out_score, fl);
    else if (lds && D < 48)
        launch_sweep<K, 48, true, false>(grid, lds_bytes, st, sn, t, rq, hotr, lead_lam, spt, n_scen, bidx, bsc, k,
                                         out_idx, out_score, fl);
    else if (lds)
        launch_sweep<K, 64, true, false>(grid, lds_bytes, st, sn, t, rq, hotr, lead_lam, spt, n_scen, bidx, bsc, k,
                                         out_idx, out_score, fl);
    else
        launch_sweep<K, 64, false, false>(grid, 0, st, sn, t, rq, hotr, lead_lam, spt, n_scen, bidx, bsc, k, out_idx,
                                          out_score, fl);
}

}  // namespace

// ------------------------------------------------------------------ no-allocation scratch
//
// Work buffers of netkv_select_batch_noalloc: one array per device in the
// code object's zero-initialised data, held until the process ends.  In
// host code its name stands for a host-side shadow, not a device address:
// the address on each device is resolved once, with that device current
// (netkv_create), and only that address is used.

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint8_t *g_scratch_dev[kMaxDevices] = {};

// Called with `device` current.
hipError_t resolve_scratch(int device) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_dev[device]) return hipSuccess;
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_dev[device] = (uint8_t *)p;
    return hipSuccess;
}

uint8_t *scratch_of(int device) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return g_scratch_dev[device];
}
}  // namespace

// ------------------------------------------------------------------ API

// ---- for the library's other translation units (netkv_internal.h)

netkv_status netkv_internal_fail(netkv_handle h, netkv_status st, const char *msg) { return fail(h, st, "%s", msg); }

void netkv_internal_clear(netkv_handle h) { h->err.clear(); }

int netkv_internal_device(netkv_handle h) { return h->device; }

uint32_t *netkv_internal_errword(netkv_handle h) { return h->errword; }

void netkv_internal_side(netkv_handle h, hipStream_t *side, hipEvent_t *fork, hipEvent_t *join) {
    *side = h->side;
    *fork = h->ev_inv_fork;
    *join = h->ev_inv_join;
}

hipError_t netkv_internal_flow_buffer(netkv_handle h, uint64_t bytes, void **out) {
    if (bytes > h->flow_buf_bytes) {
        if (h->flow_buf) (void)hipFree(h->flow_buf);
        h->flow_buf = nullptr;
        h->flow_buf_bytes = 0;
        const hipError_t e = hipMalloc(&h->flow_buf, bytes);
        if (e != hipSuccess) return e;
        h->flow_buf_bytes = bytes;
    }
    *out = h->flow_buf;
    return hipSuccess;
}

extern "C" {

netkv_status netkv_create(netkv_handle *out, int device) {
    if (!out) return NETKV_EINVAL;
    *out = nullptr;
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n) return NETKV_EINVAL;
    if (device >= kMaxDevices) return NETKV_EINVAL;
    netkv_handle h = new netkv_ctx();
    h->device = device;
    DeviceGuard g(device);
    if (resolve_scratch(device) != hipSuccess || dalloc(h->errword, 1) != hipSuccess ||
        dalloc(h->loadword, 1 + 2 * kSpreadP * kSpreadWords) != hipSuccess || hipStreamCreateWithFlags(&h->side, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&h->ev_fork0, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&h->ev_fork1, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&h->ev_join, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&h->ev_inv_fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&h->ev_inv_join, hipEventDisableTiming) != hipSuccess ||
        hipMemset(h->errword, 0, 4) != hipSuccess || hipMemset(h->loadword, 0, 4) != hipSuccess) {
        netkv_destroy(h);
        return NETKV_EDEVICE;
    }
    *out = h;
    return NETKV_OK;
}

void netkv_destroy(netkv_handle h) {
    if (!h) return;
    {
        DeviceGuard g(h->device);
        (void)hipDeviceSynchronize();
        if (h->side) (void)hipStreamDestroy(h->side);
        if (h->flow_buf) (void)hipFree(h->flow_buf);
        if (h->ev_fork0) (void)hipEventDestroy(h->ev_fork0);
        if (h->ev_fork1) (void)hipEventDestroy(h->ev_fork1);
        if (h->ev_join) (void)hipEventDestroy(h->ev_join);
        if (h->ev_inv_fork) (void)hipEventDestroy(h->ev_inv_fork);
        if (h->ev_inv_join) (void)hipEventDestroy(h->ev_inv_join);
        dfree(h->tier_map);
        dfree(h->util);
        dfree(h->n_inflight);
        dfree(h->free_mem);
        dfree(h->queue);
        dfree(h->batch);
        dfree(h->adm_prev);
        free_spare(h->spare);
        dfree(h->sl);
        dfree(h->dbase);
        dfree(h->dxlim);
        dfree(h->table);
        dfree(h->tvals);
        dfree(h->bits);
        dfree(h->sh_tab);
        dfree(h->load_buf);
        dfree(h->errword);
        dfree(h->loadword);
        dfree(h->spt_scen);
        dfree(h->dlam);
        dfree(h->bnd_lo); dfree(h->bnd_lo2); dfree(h->bnd_xm); dfree(h->bnd_xg); dfree(h->match_m);
        dfree(h->base_idx);
        dfree(h->base_score);
        dfree(h->cnt);
        dfree(h->adm);
        dfree(h->bytes);
        free_scratch(h->sc);
        dfree(h->seq_keys); dfree(h->seq_vals); dfree(h->seq_keys_out); dfree(h->seq_perm);
        dfree(h->seq_start); dfree(h->seq_end);
        for (hipEvent_t ev : h->tev) (void)hipEventDestroy(ev);
        dfree(h->rt1); dfree(h->rt2); dfree(h->ru1); dfree(h->ru2); dfree(h->sr);
    }
    delete h;
}

const char *netkv_last_error(netkv_handle h) { return h ? h->err.c_str() : "NULL handle"; }

netkv_status netkv_oracle_load(netkv_handle h, const netkv_oracle_t *o, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (!o) return fail(h, NETKV_EINVAL, "oracle is NULL");
    const uint32_t P = o->n_prefill, D = o->n_decode;
    if (P == 0 || D == 0) return fail(h, NETKV_EINVAL, "n_prefill and n_decode must be >= 1");
    if (D >= (1u << 28) || (uint64_t)P * sl_pitch(D) * 8 >= (1ull << 32))
        return fail(h, NETKV_EINVAL, "n_prefill * (n_decode + 32) must be < 2^29");
    if (!o->tier_map || !o->util || !o->n_inflight || !o->free_mem || !o->queue_depth || !o->batch_size)
        return fail(h, NETKV_EINVAL, "oracle arrays must not be NULL");
    for (int i = 0; i < 4; ++i) {
        if (!(std::isfinite(o->tier_bw[i]) && o->tier_bw[i] > 0.0))
            return fail(h, NETKV_EINVAL, "tier_bw[%d] must be finite and > 0", i);
        if (!finite_nonneg(o->tier_lat[i])) return fail(h, NETKV_EINVAL, "tier_lat[%d] must be >= 0", i);
    }
    if (!finite_nonneg(o->t_iter_a) || !finite_nonneg(o->t_iter_b) || !finite_nonneg(o->alpha))
        return fail(h, NETKV_EINVAL, "t_iter_a, t_iter_b and alpha must be finite and >= 0");
    if (o->block_tokens == 0) return fail(h, NETKV_EINVAL, "block_tokens must be >= 1");
    if (o->kv_bytes_per_token >= (1ull << 32)) return fail(h, NETKV_EINVAL, "kv_bytes_per_token >= 2^32");
    if (h->have_cache && h->cache_D != D)
        return fail(h, NETKV_EINVAL, "snapshot has %u decodes, loaded cache %u", D, h->cache_D);
    DeviceGuard g(h->device);
    hipStream_t st = (hipStream_t)stream;
    const uint64_t npd = (uint64_t)P * D;
    // stage into the spare buffers, validate, then exchange.  The wait is
    // for the whole device: selections on other streams may still read the
    // buffers exchanged out here, which the next load overwrites.
    netkv_ctx::SnapBuf &sp = h->spare;
    if (netkv_status es = ensure_spare(h, P, D)) return es;
    hipError_t e = hipSuccess;
    LoadBack back;
    const bool routes = h->have_route && h->P == P && h->D == D;   // (of another shape they are dropped below)
    if (on_device(h, o->tier_map) && on_device(h, o->util) && on_device(h, o->n_inflight) &&
        on_device(h, o->free_mem) && on_device(h, o->queue_depth) && on_device(h, o->batch_size)) {
        const SnapIn in{o->tier_map, o->util, o->n_inflight, o->free_mem, o->queue_depth, o->batch_size};
        e = hipMemsetAsync(h->loadword, 0, 4, st);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(load_snapshot_kernel,
                               dim3(grid_for(std::max<uint64_t>(npd, std::max(4u * P, D)), 256, 4096)), dim3(256), 0, st,
                               in, npd, P, D, o->beta_max, sp.tier_map, sp.util, sp.n_inflight, sp.free_mem,
                               sp.adm_prev, sp.queue, sp.batch, h->loadword);
            e = hipGetLastError();
        }
    } else {
        e = hipMemcpyAsync(sp.tier_map, o->tier_map, npd, hipMemcpyDefault, st);
        if (e == hipSuccess) e = hipMemcpyAsync(sp.util, o->util, npd * 4, hipMemcpyDefault, st);
        if (e == hipSuccess) e = hipMemcpyAsync(sp.n_inflight, o->n_inflight, 8ull * P, hipMemcpyDefault, st);
        if (e == hipSuccess) e = hipMemcpyAsync(sp.free_mem, o->free_mem, 8ull * D, hipMemcpyDefault, st);
        if (e == hipSuccess) e = hipMemcpyAsync(sp.queue, o->queue_depth, 4ull * D, hipMemcpyDefault, st);
        if (e == hipSuccess) e = hipMemcpyAsync(sp.batch, o->batch_size, 4ull * D, hipMemcpyDefault, st);
        if (e == hipSuccess) e = hipMemsetAsync(sp.adm_prev, 0, 8ull * D, st);
        if (e == hipSuccess) e = hipMemsetAsync(h->loadword, 0, 4, st);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(check_snapshot_kernel, dim3(grid_for(std::max<uint64_t>(npd, D), 256, 4096)), dim3(256),
                               0, st, sp.tier_map, sp.util, npd, sp.batch, D, o->beta_max, h->loadword);
            e = hipGetLastError();
        }
    }
    if (e == hipSuccess) {
        Snap sn{};
        sn.tier_map = sp.tier_map;
        sn.util = sp.util;
        sn.n_inflight = sp.n_inflight;
        sn.free_mem = sp.free_mem;
        sn.queue = sp.queue;
        sn.batch = sp.batch;
        for (int i = 0; i < 4; ++i) {
            sn.bw[i] = (float)o->tier_bw[i];
            sn.lat[i] = (float)o->tier_lat[i];
        }
        sn.t_a = (float)o->t_iter_a;
        sn.t_b = (float)o->t_iter_b;
        sn.alpha = (float)o->alpha;
        sn.beta_max = o->beta_max;
        sn.m_min = o->m_min;
        sn.bpt = (uint32_t)o->kv_bytes_per_token;
        sn.P = P;
        sn.D = D;
        sn.policy = h->policy_opt;
        e = launch_spread(h, sn, true, routes, h->rt1, h->ru1, h->rt2, h->ru2, st);
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&back, h->loadword, back_bytes(D, routes), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    const uint32_t bad = back.bad;
    if (e != hipSuccess) return fail(h, NETKV_EDEVICE, "snapshot upload failed: %s", hipGetErrorString(e));
    if (bad)
        return fail(h, NETKV_EINVAL, "invalid snapshot:%s%s%s", (bad & 1) ? " tier_map value > 3" : "",
                    (bad & 2) ? " util outside [0,1) or NaN" : "", (bad & 4) ? " batch_size > beta_max" : "");
    if (!h->have_snap || h->P != P || h->D != D) {
        dfree(h->sl); dfree(h->dbase); dfree(h->dxlim);
        dfree(h->bnd_lo); dfree(h->bnd_lo2); dfree(h->bnd_xm); dfree(h->bnd_xg);
        // route maps and rows of another shape no longer apply
        dfree(h->rt1); dfree(h->rt2); dfree(h->ru1); dfree(h->ru2); dfree(h->sr);
        h->rt1 = h->rt2 = nullptr;
        h->ru1 = h->ru2 = nullptr;
        h->have_route = false;
        h->have_snap = false;
        if (dalloc(h->sl, (uint64_t)P * sl_pitch(D) + kRowPad) != hipSuccess || dalloc(h->dbase, D) != hipSuccess ||
            dalloc(h->dxlim, D) != hipSuccess)
            return fail(h, NETKV_ENOMEM, "snapshot allocation failed");
        const uint32_t ng = (D + kWave - 1) / kWave;
        if (bound_pool(D) && (dalloc(h->bnd_lo, (uint64_t)P * ng) != hipSuccess ||
                              dalloc(h->bnd_lo2, (uint64_t)P * ng) != hipSuccess ||
                              dalloc(h->bnd_xm, (uint64_t)ng * kWave) != hipSuccess || dalloc(h->bnd_xg, ng) != hipSuccess))
            return fail(h, NETKV_ENOMEM, "bound table allocation failed");
    }
    std::swap(h->tier_map, sp.tier_map);
    std::swap(h->util, sp.util);
    std::swap(h->n_inflight, sp.n_inflight);
    std::swap(h->free_mem, sp.free_mem);
    std::swap(h->adm_prev, sp.adm_prev);
    std::swap(h->queue, sp.queue);
    std::swap(h->batch, sp.batch);
    // the buffers exchanged out are the next load's if they have this shape
    if (h->P != P || h->D != D) free_spare(sp);
    h->P = P;
    h->D = D;
    for (int i = 0; i < 4; ++i) {
        h->bw[i] = (float)o->tier_bw[i];
        h->bw64[i] = o->tier_bw[i];
        h->lat[i] = (float)o->tier_lat[i];
    }
    h->t_a = (float)o->t_iter_a;
    h->t_b = (float)o->t_iter_b;
    h->alpha = (float)o->alpha;
    h->beta_max = o->beta_max;
    h->m_min = o->m_min;
    h->bpt = (uint32_t)o->kv_bytes_per_token;
    h->block_tokens = o->block_tokens;
    h->have_snap = true;
    read_spread(h, P, false, back);
    if (routes) read_spread(h, P, true, back);
    return NETKV_OK;
}

netkv_status netkv_oracle_set_util(netkv_handle h, const float *util, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (!h->have_snap) return fail(h, NETKV_ENOTREADY, "no snapshot loaded");
    if (!util) return fail(h, NETKV_EINVAL, "util is NULL");
    DeviceGuard g(h->device);
    hipStream_t st = (hipStream_t)stream;
    const uint64_t npd = (uint64_t)h->P * h->D;
    // staged in the spare snapshot's matrix, then exchanged (the wait is for the
    // whole device, as in netkv_oracle_load)
    if (netkv_status es = ensure_spare(h, h->P, h->D)) return es;
    float *ut = h->spare.util;
    uint32_t bad = 0;
    hipError_t e = hipMemcpyAsync(ut, util, npd * 4, hipMemcpyDefault, st);
    if (e == hipSuccess) e = hipMemsetAsync(h->loadword, 0, 4, st);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(check_snapshot_kernel, dim3(grid_for(npd, 256, 4096)), dim3(256), 0, st,
                           (const uint8_t *)nullptr, ut, npd, (const uint32_t *)nullptr, 0u, 0u, h->loadword);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&bad, h->loadword, 4, hipMemcpyDeviceToHost, st);
    const hipError_t e2 = hipDeviceSynchronize();
    if (e == hipSuccess) e = e2;
    if (e != hipSuccess || bad)
        return e != hipSuccess ? fail(h, NETKV_EDEVICE, "util upload failed: %s", hipGetErrorString(e))
                               : fail(h, NETKV_EINVAL, "invalid util: values outside [0,1) or NaN");
    std::swap(h->util, h->spare.util);
    return NETKV_OK;
}

netkv_status netkv_congestion_smooth(netkv_handle h, const float *obs, float beta, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (!h->have_snap) return fail(h, NETKV_ENOTREADY, "no snapshot loaded");
    if (!obs) return fail(h, NETKV_EINVAL, "obs is NULL");
    if (!(beta > 0.0f && beta <= 1.0f)) return fail(h, NETKV_EINVAL, "beta must be in (0, 1]");
    DeviceGuard g(h->device);
    hipStream_t st = (hipStream_t)stream;
    const uint64_t npd = (uint64_t)h->P * h->D;
    HIPCHK(h, time_begin(h, st));
    if (((uintptr_t)obs & 15) == 0 && ((uintptr_t)h->util & 15) == 0)
        hipLaunchKernelGGL(smooth_kernel<true>, dim3(grid_for((npd + 3) / 4, 256, 8192)), dim3(256), 0, st, h->util,
                           obs, npd, beta, h->errword);
    else
        hipLaunchKernelGGL(smooth_kernel<false>, dim3(grid_for(npd, 256, 8192)), dim3(256), 0, st, h->util, obs,
                           npd, beta, h->errword);
    HIPCHK(h, hipGetLastError());
    HIPCHK(h, time_end(h, st));
    return NETKV_OK;
}

netkv_status netkv_congestion_get(netkv_handle h, float *out, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (!h->have_snap) return fail(h, NETKV_ENOTREADY, "no snapshot loaded");
    if (!out) return fail(h, NETKV_EINVAL, "out is NULL");
    DeviceGuard g(h->device);
    HIPCHK(h, hipMemcpyAsync(out, h->util, (uint64_t)h->P * h->D * sizeof(float), hipMemcpyDeviceToDevice,
                             (hipStream_t)stream));
    return NETKV_OK;
}

netkv_status netkv_route2_load(netkv_handle h, const uint8_t *tier1, const float *util1, const uint8_t *tier2,
                               const float *util2, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (!h->have_snap) return fail(h, NETKV_ENOTREADY, "no snapshot loaded");
    if (!tier1 || !util1 || !tier2 || !util2) return fail(h, NETKV_EINVAL, "a route map is NULL");
    DeviceGuard g(h->device);
    hipStream_t st = (hipStream_t)stream;
    const uint64_t npd = (uint64_t)h->P * h->D;
    uint8_t *a = nullptr, *b = nullptr;
    float *ua = nullptr, *ub = nullptr;
    auto drop = [&]() { dfree(a); dfree(b); dfree(ua); dfree(ub); };
    if (dalloc(a, npd) != hipSuccess || dalloc(b, npd) != hipSuccess || dalloc(ua, npd) != hipSuccess ||
        dalloc(ub, npd) != hipSuccess || (!h->sr && dalloc(h->sr, (uint64_t)h->P * sl_pitch(h->D) + kRowPad) != hipSuccess)) {
        drop();
        return fail(h, NETKV_ENOMEM, "route map allocation failed");
    }
    LoadBack back;
    hipError_t e = hipMemcpyAsync(a, tier1, npd, hipMemcpyDefault, st);
    if (e == hipSuccess) e = hipMemcpyAsync(b, tier2, npd, hipMemcpyDefault, st);
    if (e == hipSuccess) e = hipMemcpyAsync(ua, util1, npd * 4, hipMemcpyDefault, st);
    if (e == hipSuccess) e = hipMemcpyAsync(ub, util2, npd * 4, hipMemcpyDefault, st);
    if (e == hipSuccess) e = hipMemsetAsync(h->loadword, 0, 4, st);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(check_snapshot_kernel, dim3(grid_for(npd, 256, 4096)), dim3(256), 0, st,
                           (const uint8_t *)a, (const float *)ua, npd, (const uint32_t *)nullptr, 0u, 0u,
                           h->loadword);
        hipLaunchKernelGGL(check_snapshot_kernel, dim3(grid_for(npd, 256, 4096)), dim3(256), 0, st,
                           (const uint8_t *)b, (const float *)ub, npd, (const uint32_t *)nullptr, 0u, 0u,
                           h->loadword);
        e = launch_spread(h, make_snap(h), false, true, a, ua, b, ub, st);
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&back, h->loadword, back_bytes(h->D, true), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    const uint32_t bad = back.bad;
    if (e != hipSuccess || bad) {
        drop();
        return e != hipSuccess ? fail(h, NETKV_EDEVICE, "route map upload failed: %s", hipGetErrorString(e))
                               : fail(h, NETKV_EINVAL, "invalid route map:%s%s", (bad & 1) ? " tier value > 3" : "",
                                      (bad & 2) ? " util outside [0,1) or NaN" : "");
    }
    dfree(h->rt1);
    dfree(h->rt2);
    dfree(h->ru1);
    dfree(h->ru2);
    h->rt1 = a;
    h->rt2 = b;
    h->ru1 = ua;
    h->ru2 = ub;
    h->have_route = true;
    read_spread(h, h->P, true, back);
    return NETKV_OK;
}

netkv_status netkv_route2_clear(netkv_handle h) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    DeviceGuard g(h->device);
    dfree(h->rt1);
    dfree(h->rt2);
    dfree(h->ru1);
    dfree(h->ru2);
    h->rt1 = h->rt2 = nullptr;
    h->ru1 = h->ru2 = nullptr;
    h->have_route = false;
    return NETKV_OK;
}

netkv_status netkv_route2_of(netkv_handle h, const netkv_requests_t *req, uint32_t k, const int32_t *idx,
                             int8_t *out_route, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    netkv_status st = check_requests(h, req);
    if (st) return st;
    if (k < 1 || k > 8) return fail(h, NETKV_EINVAL, "k must be in [1, 8]");
    if (req->n_req && (!idx || !out_route)) return fail(h, NETKV_EINVAL, "idx and out_route must not be NULL");
    if ((st = ready(h))) return st;
    if (!h->have_route) return fail(h, NETKV_ENOTREADY, "no route maps loaded (netkv_route2_load)");
    if (req->n_req == 0) return NETKV_OK;
    DeviceGuard g(h->device);
    hipStream_t s = (hipStream_t)stream;
    Snap sn = make_snap(h);
    const uint64_t nd = std::max<uint64_t>((uint64_t)h->P * h->D, h->D);
    hipLaunchKernelGGL(derive_kernel, dim3((uint32_t)((nd + 255) / 256)), dim3(256), 0, s, sn, h->sl, h->dbase,
                       h->dxlim);
    hipLaunchKernelGGL(derive_route_kernel, dim3((uint32_t)((nd + 255) / 256)), dim3(256), 0, s, sn,
                       (const uint8_t *)h->rt1, (const float *)h->ru1, (const uint8_t *)h->rt2,
                       (const float *)h->ru2, h->sr);
    sn.sr = h->sr;
    const uint64_t n = (uint64_t)req->n_req * k;
    hipLaunchKernelGGL(route_of_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, sn, make_table(h),
                       make_reqs(req), k, idx, out_route);
    HIPCHK(h, hipGetLastError());
    return NETKV_OK;
}

netkv_status netkv_selection_bytes(netkv_handle h, const netkv_requests_t *req, uint32_t k, const int32_t *idx,
                                   uint64_t *out_bytes, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    netkv_status st = check_requests(h, req);
    if (st) return st;
    if (k < 1 || k > 8) return fail(h, NETKV_EINVAL, "k must be in [1, 8]");
    if (req->n_req && (!idx || !out_bytes)) return fail(h, NETKV_EINVAL, "idx and out_bytes must not be NULL");
    if ((st = ready(h))) return st;
    if (req->n_req == 0) return NETKV_OK;
    DeviceGuard g(h->device);
    const uint64_t n = (uint64_t)req->n_req * k;
    hipLaunchKernelGGL(selection_bytes_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       make_snap(h), make_table(h), make_reqs(req), k, idx, out_bytes, h->errword);
    HIPCHK(h, hipGetLastError());
    return NETKV_OK;
}

netkv_status netkv_cache_load(netkv_handle h, uint32_t n_decode, const uint64_t *hash_off, const uint64_t *hashes,
                              uint64_t n_hashes, float max_load_factor, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (n_decode == 0 || !hash_off) return fail(h, NETKV_EINVAL, "n_decode must be >= 1 and hash_off non-NULL");
    if (n_hashes && !hashes) return fail(h, NETKV_EINVAL, "hashes is NULL");
    if (!(max_load_factor > 0.0f && max_load_factor < 1.0f))
        return fail(h, NETKV_EINVAL, "max_load_factor must be in (0, 1)");
    if (h->have_snap && h->D != n_decode)
        return fail(h, NETKV_EINVAL, "cache has %u decodes, loaded snapshot %u", n_decode, h->D);
    DeviceGuard g(h->device);
    hipStream_t st = (hipStream_t)stream;
    std::vector<uint64_t> off(n_decode + 1);
    HIPCHK(h, hipMemcpyAsync(off.data(), hash_off, 8ull * (n_decode + 1), hipMemcpyDefault, st));
    HIPCHK(h, hipStreamSynchronize(st));
    for (uint32_t d = 0; d < n_decode; ++d)
        if (off[d + 1] < off[d]) return fail(h, NETKV_EINVAL, "hash_off decreases at decode %u", d);
    if (off[n_decode] > n_hashes) return fail(h, NETKV_EINVAL, "hash_off[n_decode] exceeds n_hashes");
    const uint64_t first = off[0], total = off[n_decode] - off[0];
    if (total >= (1ull << 31)) return fail(h, NETKV_ECAPACITY, "more than 2^31 - 1 resident hashes");
    // words per holder bitmap row: whole 64-decode words, rounded up to a
    // multiple of 12 so that every decodes-per-lane choice C (1, 2, 3, 4, 6)
    // reads its groups' C words inside the row, at 8 * C-byte alignment
    const uint64_t bwords = ((uint64_t)n_decode + 63) / 64;
    const uint32_t bpitch = (uint32_t)((bwords + 11) / 12 * 12);
    // two slots per bucket; two-choice cuckoo sets of 2-slot buckets can be
    // built up to an occupancy of about 0.897, and are capped at 0.85
    const double lf = std::min(0.85, (double)max_load_factor);
    auto log2_buckets = [&](uint64_t n, double f) {
        const double need = std::ceil((double)n / (2.0 * f));
        uint32_t b = 3;
        while (b < 40 && (double)(1ull << b) < need) ++b;
        return b;
    };
    // parts that would fill 2^11 buckets each if every hash were distinct, or
    // 2^12 where those would be more than two sort passes of 8 bits can tell
    // apart (with 160 KiB of LDS per CU, 3 or 1 workgroups work on a CU)
    const uint32_t most = log2_buckets(total, std::max(lf, 0.5));
    const bool big = most > 16 + kBlockLog2;
    const uint32_t part_lg = kBlockLog2 + (big ? 1 : 0);
    const uint32_t bits = most > part_lg ? most - part_lg : 0u;   // at most 19: total < 2^31
    const uint32_t n_part = 1u << bits;
    size_t tb = 0;
    if (total && bits)
        HIPCHK(h, rocprim::radix_sort_pairs(nullptr, tb, (const uint64_t *)nullptr, (uint64_t *)nullptr,
                                            (const uint32_t *)nullptr, (uint32_t *)nullptr, (uint32_t)total,
                                            0, bits, st));
    // work buffer: the pairs twice (the sort's input, which then takes the
    // distinct hashes, and its output), offsets, parts, counters
    uint64_t at = 0;
    auto take = [&](uint64_t bytes) {
        const uint64_t o = at;
        at += (bytes + 255) / 256 * 256;
        return o;
    };
    const uint64_t o_key = take(8 * total), o_key2 = take(8 * total), o_dec = take(4 * total), o_dec2 = take(4 * total);
    const uint64_t o_off = take(8ull * (n_decode + 1)), o_start = take(4ull * (n_part + 1)), o_count = take(4ull * n_part);
    const uint64_t o_cnt = take(24), o_tmp = take(std::max<size_t>(tb, 16));
    uint8_t *buf = h->load_buf;
    if (at > h->load_bytes) {
        dfree(h->load_buf);
        h->load_bytes = 0;
        if (dalloc(h->load_buf, at) != hipSuccess) return fail(h, NETKV_ENOMEM, "staging allocation failed");
        buf = h->load_buf;
        h->load_bytes = at;
    }
    // a work buffer of up to kLoadKeep bytes stays for the next load
    struct Drop {
        netkv_handle h;
        ~Drop() {
            if (h->load_bytes > kLoadKeep) {
                dfree(h->load_buf);
                h->load_bytes = 0;
            }
        }
    } drop{h};
    uint64_t *key = (uint64_t *)(buf + o_key), *key2 = (uint64_t *)(buf + o_key2), *doff = (uint64_t *)(buf + o_off);
    uint32_t *dec = (uint32_t *)(buf + o_dec), *dec2 = (uint32_t *)(buf + o_dec2);
    uint32_t *start = (uint32_t *)(buf + o_start), *count = (uint32_t *)(buf + o_count);
    struct Counters {
        unsigned long long n[2];   // distinct hashes, those of several holders
        uint32_t rows, flag;       // next bitmap row; errors
    } c{};
    Counters *dc = (Counters *)(buf + o_cnt);
    c.rows = 1;   // row 0: all zero
    hipError_t e = hipMemcpyAsync(doff, off.data(), 8ull * (n_decode + 1), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(dc, &c, sizeof c, hipMemcpyHostToDevice, st);
    if (e == hipSuccess && total) {
        const uint64_t *src = hashes + first;
        if (!on_device(h, hashes)) {
            e = hipMemcpyAsync(key, src, 8ull * total, hipMemcpyDefault, st);
            src = key;
        }
        if (e == hipSuccess) {
            hipLaunchKernelGGL(pair_kernel, dim3((uint32_t)((total + kBlock * kPairPer - 1) / (kBlock * kPairPer))),
                               dim3(kBlock), 0, st, (const uint64_t *)doff, n_decode, first, total, src, bits, key,
                               dec, &dc->flag);
            e = hipGetLastError();
        }
        if (e == hipSuccess && bits)
            e = rocprim::radix_sort_pairs(buf + o_tmp, tb, (const uint64_t *)key, key2, (const uint32_t *)dec, dec2,
                                          (uint32_t)total, 0, bits, st);
        if (e == hipSuccess && !bits) {   // one part: the pairs as they are
            std::swap(key, key2);
            std::swap(dec, dec2);
        }
        if (e == hipSuccess) {
            hipLaunchKernelGGL(parts_kernel, dim3((uint32_t)(total / 256 + 1)), dim3(256), 0, st,
                               (const uint64_t *)key2, total, bits, start);
            if (big)
                hipLaunchKernelGGL((dedupe_kernel<2 * kBlockSlots>), dim3(n_part), dim3(1024), 0, st,
                                   (const uint64_t *)key2, (const uint32_t *)dec2, (const uint32_t *)start, bits, key, dec,
                                   count, dc->n, &dc->flag);
            else
                hipLaunchKernelGGL((dedupe_kernel<kBlockSlots>), dim3(n_part), dim3(512), 0, st,
                                   (const uint64_t *)key2, (const uint32_t *)dec2, (const uint32_t *)start, bits, key, dec,
                                   count, dc->n, &dc->flag);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipMemcpyAsync(&c, dc, sizeof c, hipMemcpyDeviceToHost, st);
    }
    {
        // (also after an error: the host's copies end here; the device, since
        // selections on other streams may still read the index whose buffers
        // are reused below)
        const hipError_t e2 = hipDeviceSynchronize();
        if (e == hipSuccess) e = e2;
    }
    if (e != hipSuccess) return fail(h, NETKV_EDEVICE, "index build failed: %s", hipGetErrorString(e));
    if (c.flag & 1u) return fail(h, NETKV_EINVAL, "cache contains the reserved hash value 0");
    // the whole set's pairs: sorted by all bits, once; then key / dec hold them
    bool whole = false;
    auto sort_whole = [&]() -> netkv_status {
        if (whole) return NETKV_OK;
        whole = true;
        size_t wb = 0;
        HIPCHK(h, rocprim::radix_sort_pairs(nullptr, wb, (const uint64_t *)key2, key, (const uint32_t *)dec2, dec,
                                            (uint32_t)total, 0, 64, st));
        uint8_t *tmp = buf + o_tmp, *own = nullptr;
        if (wb > std::max<size_t>(tb, 16)) {
            if (dalloc(own, wb) != hipSuccess) return fail(h, NETKV_ENOMEM, "sort scratch allocation failed");
            tmp = own;
        }
        hipError_t e = rocprim::radix_sort_pairs(tmp, wb, (const uint64_t *)key2, key, (const uint32_t *)dec2, dec,
                                                 (uint32_t)total, 0, 64, st);
        Counters z{};
        z.rows = 1;
        if (e == hipSuccess) e = hipMemcpyAsync(dc, &z, sizeof z, hipMemcpyHostToDevice, st);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(whole_count_kernel, dim3(grid_for(total, 256, 16384)), dim3(256), 0, st,
                               (const uint64_t *)key, (const uint32_t *)dec, total, dc->n);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipMemcpyAsync(&c, dc, sizeof c, hipMemcpyDeviceToHost, st);
        const hipError_t e2 = hipStreamSynchronize(st);   // (the buffer's uses end here)
        if (e == hipSuccess) e = e2;
        dfree(own);
        if (e != hipSuccess) return fail(h, NETKV_EDEVICE, "index build failed: %s", hipGetErrorString(e));
        return NETKV_OK;
    };
    netkv_status ns;
    if (c.flag && (ns = sort_whole())) return ns;   // a part was too full
    const uint64_t distinct = c.n[0], rows = c.n[1] + 1;   // row 0: all zero
    if (rows >= (uint64_t)kHeldOne)
        return fail(h, NETKV_ECAPACITY, "more than 2^31 - 2 hashes held by several decodes");
    const uint32_t planned = log2_buckets(distinct, lf);
    if (planned > 30) return fail(h, NETKV_ECAPACITY, "the index would need more than 2^31 slots");
    // a blocked set beyond kBlockedMost takes twice the buckets, or is a whole
    // one where the set can have no more
    uint32_t log2b = planned;
    if (!whole && planned > kBlockLog2 && (double)distinct > kBlockedMost * 2.0 * (double)(1ull << planned)) {
        if (planned < 30) ++log2b;
        else if ((ns = sort_whole())) return ns;
    }
    // the old index is given up here; its buffers serve the new one where they
    // have its size (else they are released first: the new one may be large)
    h->have_cache = false;
    const uint64_t row_words = rows * bpitch;
    if (row_words > h->bits_cap || row_words < h->bits_cap / 2) {
        dfree(h->bits);
        h->bits_cap = 0;
    }
    const bool shared = rows > 1 && rows <= kSharedMaxRows;
    uint32_t lb = 3;
    while ((1ull << lb) < 3 * rows) ++lb;
    if (h->sh_log2b != lb || !shared) dfree(h->sh_tab);
    auto drop_table = [&]() {
        dfree(h->table);
        dfree(h->tvals);
        h->log2b = 0;
    };
    auto take_table = [&]() {   // 2^log2b buckets
        if (h->log2b != log2b) drop_table();
        if (h->table && h->tvals) return true;
        if (dalloc(h->table, 2ull << log2b) != hipSuccess || dalloc(h->tvals, 2ull << log2b) != hipSuccess) {
            (void)hipGetLastError();
            drop_table();
            return false;
        }
        h->log2b = log2b;
        return true;
    };
    if (h->log2b != log2b) drop_table();
    if (!h->bits) {
        if (dalloc(h->bits, row_words) != hipSuccess)
            return fail(h, NETKV_ENOMEM, "holder bitmap allocation of %llu bytes failed",
                        (unsigned long long)(8 * row_words));
        h->bits_cap = row_words;
    }
    // should a blocked build fail to place every key (a random walk that did
    // not end), or have no memory for twice the buckets, the set is built
    // whole at the planned size, and where that fails with twice the buckets,
    // twice
    for (int attempt = 0;;) {
        if (!take_table()) {
            if (!whole && log2b > planned) {
                if ((ns = sort_whole())) return ns;
                log2b = planned;
                continue;
            }
            return fail(h, NETKV_ENOMEM, "index allocation of %llu bytes failed", (unsigned long long)(24ull << log2b));
        }
        // the shared index; without it (too many shared hashes to stay in
        // cache, a whole set, whose hashes may crowd in few slots, no memory)
        // lookups go to the set
        if (whole) dfree(h->sh_tab);
        else if (shared && !h->sh_tab) {
            if (dalloc(h->sh_tab, 1ull << lb) != hipSuccess) (void)hipGetLastError();
            h->sh_log2b = lb;
        }
        const uint64_t nbk = 1ull << log2b;
        c.rows = 1;
        c.flag = 0;
        e = hipMemsetAsync(h->bits, 0, 8 * row_words, st);
        if (e == hipSuccess && h->sh_tab) e = hipMemsetAsync(h->sh_tab, 0, 16ull << lb, st);
        if (e == hipSuccess && (whole || !total)) e = hipMemsetAsync(h->table, 0, 16 * nbk, st);
        if (e == hipSuccess) e = hipMemcpyAsync(dc, &c, sizeof c, hipMemcpyHostToDevice, st);
        const uint32_t lg = std::min(log2b, std::max(kBlockLog2, std::min(part_lg, log2b > bits ? log2b - bits : 0u)));
        Build u{key2, dec2, key, dec, start, count, bits, lg, log2b, h->table, h->tvals, h->bits, bpitch,
                h->sh_tab, 64u - lb, (1u << lb) - 1u, &dc->rows, &dc->flag};
        if (e == hipSuccess && total && !whole) {
            const uint32_t grid = 1u << (log2b - lg);
            if (lg > kBlockLog2)
                hipLaunchKernelGGL((build_kernel<2 * kBlockSlots>), dim3(grid), dim3(1024), 0, st, u);
            else
                hipLaunchKernelGGL((build_kernel<kBlockSlots>), dim3(grid), dim3(512), 0, st, u);
            e = hipGetLastError();
        } else if (e == hipSuccess && total) {
            u.key = key;
            u.dec = dec;
            const dim3 grid(grid_for(total, 256, 16384));
            hipLaunchKernelGGL(whole_insert_kernel, grid, dim3(256), 0, st, u, total);
            hipLaunchKernelGGL(whole_value_kernel, grid, dim3(256), 0, st, u, total);
            hipLaunchKernelGGL(whole_unmix_kernel, dim3(grid_for(2 * nbk, 256, 16384)), dim3(256), 0, st, h->table,
                               2 * nbk);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipMemcpyAsync(&c, dc, sizeof c, hipMemcpyDeviceToHost, st);
        const hipError_t e2 = hipStreamSynchronize(st);
        if (e == hipSuccess) e = e2;
        if (e != hipSuccess || !c.flag) break;
        if (!whole) {
            if ((ns = sort_whole())) return ns;
            log2b = planned;
        } else {
            if (attempt++ == 2 || log2b >= 30) break;
            ++log2b;
        }
    }
    if (e != hipSuccess || c.flag)
        return e != hipSuccess ? fail(h, NETKV_EDEVICE, "index build failed: %s", hipGetErrorString(e))
                               : fail(h, NETKV_ECAPACITY, "index build could not place every hash");
    const uint64_t nbk = 1ull << log2b;
    h->whole = whole;
    h->buckets = nbk;
    h->bpitch = bpitch;
    h->rows = rows;
    h->distinct = distinct;
    h->table_bytes = 24 * nbk + 8 * rows * bpitch;
    h->cache_D = n_decode;
    h->have_cache = true;
    return NETKV_OK;
}

netkv_status netkv_select_batch(netkv_handle h, const netkv_requests_t *req, uint32_t k, int32_t *out_idx,
                                float *out_score, netkv_pairs_t *pairs, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    netkv_status st = check_requests(h, req);
    if (st) return st;
    if (k < 1 || k > 8) return fail(h, NETKV_EINVAL, "k must be in [1, 8]");
    if (req->n_req && (!out_idx || !out_score))
        return fail(h, NETKV_EINVAL, "out_idx and out_score must not be NULL");
    if ((st = ready(h))) return st;
    if (req->n_req == 0) return NETKV_OK;
    DeviceGuard g(h->device);
    hipStream_t s = (hipStream_t)stream;
    PairOut po{nullptr, nullptr, nullptr};
    bool want_pairs = false;
    if (pairs) {
        po.j = pairs->prefix_blocks;
        po.feas = pairs->feasible;
        po.score = pairs->score;
        want_pairs = po.j || po.feas || po.score;
    }
    if (!want_pairs && direct_batch(h, req->n_req, req->n_hashes, kDirectTasks)) {
        h->last_form = 3;
        st = run_direct(h, req, k, out_idx, out_score, s, true);
    } else if (!want_pairs && bounded_batch(h, req->n_req, req->n_hashes, k, h->have_route)) {
        h->last_form = 2;
        st = run_bounded(h, req, k, out_idx, out_score, s, true);
    } else {
        h->last_form = 1;
        st = select_owned(h, req, k, out_idx, out_score, po, want_pairs, 0xFFFFFFFFu, s, true);
    }
    if (!st) size_ahead(h, req, k, s);
    return st;
}

netkv_status netkv_select_batch_noalloc(netkv_handle h, const netkv_requests_t *req, uint32_t k, int32_t *out_idx,
                                        float *out_score, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    netkv_status st = check_requests(h, req);
    if (st) return st;
    if (k < 1 || k > 8) return fail(h, NETKV_EINVAL, "k must be in [1, 8]");
    if (req->n_req && (!out_idx || !out_score))
        return fail(h, NETKV_EINVAL, "out_idx and out_score must not be NULL");
    if ((st = ready(h))) return st;
    if (req->n_req == 0) return NETKV_OK;
    uint8_t *base = scratch_of(h->device);
    if (!base) return fail(h, NETKV_EDEVICE, "no-allocation scratch not resolved on device %d", h->device);
    DeviceGuard g(h->device);
    hipStream_t s = (hipStream_t)stream;
    Scratch sc;
    uint64_t r_sub = 0;
    if ((st = carve_static(h, base, req->n_req, k, sc, r_sub))) return st;
    const bool direct = direct_batch(h, req->n_req, req->n_hashes, kDirectTasks);
    h->last_form = direct ? 3 : 1;
    if (direct) return run_direct(h, req, k, out_idx, out_score, s, true);
    const PairOut po{nullptr, nullptr, nullptr};
    for (uint64_t r0 = 0; r0 < req->n_req; r0 += r_sub) {
        netkv_requests_t sub = *req;
        sub.n_req = (uint32_t)std::min<uint64_t>(r_sub, req->n_req - r0);
        sub.prefill += r0;
        sub.len_tokens += r0;
        sub.hash_off += r0;   // absolute offsets into the same hash array
        if ((st = run_select(h, sc, &sub, k, out_idx + r0 * k, out_score + r0 * k, po, false, 0xFFFFFFFFu, s, true,
                             r0 == 0)))
            return st;
    }
    return NETKV_OK;
}

netkv_status netkv_reserve(netkv_handle h, uint32_t max_req, uint64_t max_hashes, uint32_t max_k, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (max_k < 1 || max_k > 8) return fail(h, NETKV_EINVAL, "max_k must be in [1, 8]");
    if (max_req > (1u << 31)) return fail(h, NETKV_EINVAL, "max_req too large");
    if (!h->have_snap) return fail(h, NETKV_ENOTREADY, "no snapshot loaded (netkv_oracle_load)");
    if (max_req == 0) return NETKV_OK;
    DeviceGuard g(h->device);
    uint64_t elems = 0;
    for (uint32_t k = 1; k <= max_k; ++k) {
        const Geometry geo = geometry(h, k);
        elems = std::max<uint64_t>(elems, (uint64_t)max_req * geo.ngroup * geo.K);
    }
    netkv_status st = ensure_scratch(h, h->sc, max_req, elems, max_hashes, (hipStream_t)stream);
    if (!st) st = ensure_match(h, max_req);
    if (!st) st = ensure_hotr(h, max_req);
    if (!st) st = ensure_dlam(h, std::min<uint64_t>(max_req, kDirectRecordTasks / ((h->D + kWave - 1) / kWave)));
    if (!st) st = ensure_seq(h, max_req, h->P, true, true);
    return st;
}

netkv_status netkv_rank_sweep(netkv_handle h, const netkv_requests_t *req, uint32_t n_scen, const float *util_scen,
                              uint32_t k, int32_t *out_idx, float *out_score, uint64_t *out_flips,
                              uint64_t *out_inversions, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    netkv_status st = check_requests(h, req);
    if (st) return st;
    if (k < 1 || k > 8) return fail(h, NETKV_EINVAL, "k must be in [1, 8]");
    if (n_scen > 65535) return fail(h, NETKV_EINVAL, "n_scen must be <= 65535");
    if (n_scen && !util_scen) return fail(h, NETKV_EINVAL, "util_scen must not be NULL");
    if (n_scen && req->n_req && (!out_idx || !out_score))
        return fail(h, NETKV_EINVAL, "out_idx and out_score must not be NULL");
    if ((st = ready(h))) return st;
    if (n_scen == 0) return NETKV_OK;
    DeviceGuard g(h->device);
    hipStream_t s = (hipStream_t)stream;
    const uint64_t R = req->n_req, P = h->P, D = h->D;
    Snap sn = make_snap(h);
    if (out_flips) {
        hipLaunchKernelGGL(fill_u64_kernel, dim3(grid_for(2ull * n_scen, 256)), dim3(256), 0, s, out_flips,
                           2ull * n_scen, 0ull);
        HIPCHK(h, hipGetLastError());
    }
    // The caller's stream waits for the second stream when the call
    // returns (every path), if the counts below were forked onto it.
    struct Join {
        hipStream_t s;
        hipEvent_t e;
        bool on = false;
        ~Join() {
            if (on) (void)hipStreamWaitEvent(s, e, 0);
        }
    } join{s, h->ev_inv_join};
    if (out_inversions) {
        // Proposition 2's counts depend on the snapshot and the scenarios
        // only.  When the selection below leaves the second stream free (a
        // batch below kForkMinN requests) they run there, beside the
        // selection and the sweep.
        const bool fork = R > 0 && R < kForkMinN;
        hipStream_t si = fork ? h->side : s;
        if (fork) {
            HIPCHK(h, hipEventRecord(h->ev_inv_fork, s));
            HIPCHK(h, hipStreamWaitEvent(si, h->ev_inv_fork, 0));
        }
        hipLaunchKernelGGL(fill_u64_kernel, dim3(grid_for(3ull * n_scen, 256)), dim3(256), 0, si, out_inversions,
                           3ull * n_scen, 0ull);
        Bw64 bw;
        for (int i = 0; i < 4; ++i) bw.b[i] = h->bw64[i];
        hipLaunchKernelGGL(tier_inv_kernel, dim3((uint32_t)((P * D + 255) / 256), n_scen), dim3(256), 0, si, sn, bw,
                           util_scen, (unsigned long long *)out_inversions);
        HIPCHK(h, hipGetLastError());
        if (fork) {
            HIPCHK(h, hipEventRecord(h->ev_inv_join, si));
            join.on = true;
        }
    }
    if (R == 0) return NETKV_OK;
    if ((st = ensure_seq(h, R, P, false, true))) return st;
    const uint64_t nspt = (uint64_t)n_scen * P * D;
    if (h->spt_cap < nspt) {
        dfree(h->spt_scen);
        h->spt_cap = 0;
        HIPCHK(h, dalloc(h->spt_scen, nspt));
        h->spt_cap = nspt;
    }
    // the selection under the loaded congestion, keeping every request's
    // scoring record by batch index and the leaders' prefix lengths
    const float *lead_lam = nullptr;
    {
        TimingOff off(h);  // only the sweep kernel is timed
        const PairOut po{nullptr, nullptr, nullptr};
        // (pools of more than 64 decodes read the rows anew for every scenario, and
        // a wavefront's 64 rows of their own stay in the 32 KiB L1 up to 128
        // decodes: 16 scenarios of 4,000 requests on 192 decodes 1,122 us from the
        // batch order, 1,197 so; 63 of 89 on 120 decodes 945 and 912)
        if ((D <= 2u * kWave || n_scen <= 8) && direct_batch(h, R, req->n_hashes, kDirectRecordTasks)) {
            if ((st = ensure_hotr(h, R)) || (st = ensure_dlam(h, R))) return st;
            if ((st = run_direct(h, req, 1, h->base_idx, h->base_score, s, false, h->sc.hotr, h->dlam))) return st;
            lead_lam = h->dlam;
        } else {
            if ((st = select_owned(h, req, 1, h->base_idx, h->base_score, po, false, 0xFFFFFFFFu, s, false, true)))
                return st;
            lead_lam = h->sc.lead_lam;
        }
    }
    hipLaunchKernelGGL(derive_scen_kernel, dim3((uint32_t)((nspt + 255) / 256)), dim3(256), 0, s, sn, util_scen, nspt,
                       h->spt_scen);
    HIPCHK(h, hipGetLastError());
    const Reqs rq = make_reqs(req);
    const Table t = make_table(h);
    const uint32_t Dp = (uint32_t)D | 1u;
    const bool lds = P * Dp <= kSweepMaxTab;
    // a third table (the next scenario's) when the threads hold its entries
    const bool held = (uint64_t)P * D <= (uint64_t)kSweepThreads * kSweepHold;
    const size_t lds_bytes = lds ? (held ? 3 : 2) * P * Dp * sizeof(float) : 0;
    const dim3 grid((uint32_t)((R + kSweepThreads - 1) / kSweepThreads), (n_scen + kSweepScen - 1) / kSweepScen);
    unsigned long long *fl = (unsigned long long *)out_flips;
    HIPCHK(h, time_begin(h, s));
#define NETKV_SWEEP(KK)                                                                                            \
    launch_sweep_k<KK>((uint32_t)D, lds, grid, lds_bytes, s, sn, t, rq, h->sc.hotr, lead_lam, h->spt_scen,          \
                       n_scen, h->base_idx, h->base_score, k, out_idx, out_score, fl)
    if (k == 1) NETKV_SWEEP(1);
    else if (k == 2) NETKV_SWEEP(2);
    else if (k == 3) NETKV_SWEEP(3);
    else if (k == 4) NETKV_SWEEP(4);
    else NETKV_SWEEP(8);
#undef NETKV_SWEEP
    HIPCHK(h, hipGetLastError());
    HIPCHK(h, time_end(h, s));
    return NETKV_OK;
}

netkv_status netkv_commit_batch(netkv_handle h, const netkv_requests_t *req, const int32_t *sel, uint32_t cap,
                                uint32_t mu, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    netkv_status st = check_requests(h, req);
    if (st) return st;
    if (!sel && req->n_req) return fail(h, NETKV_EINVAL, "sel is NULL");
    if (cap > 65535) return fail(h, NETKV_EINVAL, "cap must be <= 65535");
    if ((st = ready(h))) return st;
    DeviceGuard g(h->device);
    hipStream_t s = (hipStream_t)stream;
    const uint64_t entries = 4ull * h->P + h->D;
    const uint64_t lds = 8ull * h->D + 4ull * entries;
    if (lds <= kCommitLds) {
        // sums in LDS: one row per workgroup, at most kCommitRows of them
        // (pools of up to 1,024 x 3,072 instances take 52 KiB)
        if (h->commit_P != h->P || h->commit_D != h->D) {
            dfree(h->cnt);
            dfree(h->bytes);
            h->commit_P = h->commit_D = 0;
            HIPCHK(h, dalloc(h->cnt, kCommitRows * entries));
            HIPCHK(h, dalloc(h->bytes, (uint64_t)kCommitRows * h->D));
            h->commit_P = h->P;
            h->commit_D = h->D;
        }
        const uint32_t nrow =
            (uint32_t)std::min<uint64_t>(((uint64_t)req->n_req * kMatchLanes + kCommitThreads - 1) / kCommitThreads,
                                         kCommitRows);
        if (nrow) {
            hipLaunchKernelGGL(commit_rows_kernel, dim3(nrow), dim3(kCommitThreads), (size_t)lds, s, make_snap(h),
                               make_table(h), make_reqs(req), sel, h->cnt, h->bytes, h->errword);
            HIPCHK(h, hipGetLastError());
        }
        hipLaunchKernelGGL(commit_sum_kernel, dim3((uint32_t)((entries + kWavesPerBlock - 1) / kWavesPerBlock)),
                           dim3(kBlock), 0, s, h->P, h->D, cap, mu, nrow, (const uint32_t *)h->cnt,
                           (const unsigned long long *)h->bytes, h->n_inflight, h->queue, h->free_mem, h->adm_prev);
        HIPCHK(h, hipGetLastError());
        return NETKV_OK;
    }
    if (h->commit_P != h->P || h->commit_D != h->D) {
        dfree(h->cnt);
        dfree(h->adm);
        dfree(h->bytes);
        h->commit_P = h->commit_D = 0;
        HIPCHK(h, dalloc(h->cnt, 4ull * h->P));
        HIPCHK(h, dalloc(h->adm, h->D));
        HIPCHK(h, dalloc(h->bytes, h->D));
        h->commit_P = h->P;
        h->commit_D = h->D;
    }
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(4ull * h->P, 256)), dim3(256), 0, s, h->cnt, 4ull * h->P, 0u);
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(h->D, 256)), dim3(256), 0, s, h->adm, (uint64_t)h->D, 0u);
    hipLaunchKernelGGL(fill_u64_kernel, dim3(grid_for(h->D, 256)), dim3(256), 0, s, (uint64_t *)h->bytes,
                       (uint64_t)h->D, 0ull);
    HIPCHK(h, hipGetLastError());
    if (req->n_req) {
        hipLaunchKernelGGL(commit_count_kernel, dim3((req->n_req + 255) / 256), dim3(256), 0, s, make_snap(h),
                           make_table(h), make_reqs(req), sel, h->cnt, h->adm, h->bytes, h->errword);
        HIPCHK(h, hipGetLastError());
    }
    const uint32_t n = 4u * h->P + h->D;
    hipLaunchKernelGGL(commit_apply_kernel, dim3((n + 255) / 256), dim3(256), 0, s, h->P, h->D, cap, mu,
                       (const uint32_t *)h->cnt, (const uint32_t *)h->adm, (const unsigned long long *)h->bytes,
                       h->n_inflight, h->queue, h->free_mem, h->adm_prev);
    HIPCHK(h, hipGetLastError());
    return NETKV_OK;
}

netkv_status netkv_state_get(netkv_handle h, uint16_t *n_inflight, uint32_t *queue_depth, uint64_t *free_mem,
                             uint64_t *admitted_prev, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (!h->have_snap) return fail(h, NETKV_ENOTREADY, "no snapshot loaded");
    DeviceGuard g(h->device);
    hipStream_t s = (hipStream_t)stream;
    if (n_inflight) HIPCHK(h, hipMemcpyAsync(n_inflight, h->n_inflight, 8ull * h->P, hipMemcpyDefault, s));
    if (queue_depth) HIPCHK(h, hipMemcpyAsync(queue_depth, h->queue, 4ull * h->D, hipMemcpyDefault, s));
    if (free_mem) HIPCHK(h, hipMemcpyAsync(free_mem, h->free_mem, 8ull * h->D, hipMemcpyDefault, s));
    if (admitted_prev) HIPCHK(h, hipMemcpyAsync(admitted_prev, h->adm_prev, 8ull * h->D, hipMemcpyDefault, s));
    HIPCHK(h, hipStreamSynchronize(s));
    return NETKV_OK;
}

netkv_status netkv_sync_errors(netkv_handle h, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    DeviceGuard g(h->device);
    hipStream_t s = (hipStream_t)stream;
    uint32_t e = 0;
    HIPCHK(h, hipStreamSynchronize(s));
    HIPCHK(h, hipMemcpy(&e, h->errword, 4, hipMemcpyDeviceToHost));
    HIPCHK(h, hipMemset(h->errword, 0, 4));
    if (e)
        return fail(h, NETKV_EINVAL, "input errors:%s%s%s%s%s%s",
                    (e & kErrRequest) ? " inconsistent request header" : "",
                    (e & kErrObservation) ? " congestion observation outside [0,1)" : "",
                    (e & kErrSelection) ? " selection index >= D" : "", (e & kErrTableFull) ? " table full" : "",
                    (e & kErrFlow) ? " invalid flow set" : "",
                    (e & kErrFlowStall) ? " flow simulation reached its iteration bound" : "");
    return NETKV_OK;
}

netkv_status netkv_set_timing(netkv_handle h, int enable) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (enable && h->tev.empty()) {
        DeviceGuard g(h->device);
        h->tev.assign(2 * kTimeSlots, nullptr);
        for (hipEvent_t &ev : h->tev) HIPCHK(h, hipEventCreate(&ev));
    }
    h->timing = enable != 0;
    h->tcount = 0;
    return NETKV_OK;
}

netkv_status netkv_kernel_ms(netkv_handle h, float *ms) {
    if (!h || !ms) return NETKV_EINVAL;
    h->err.clear();
    if (h->tcount == 0) return fail(h, NETKV_ENOTREADY, "no timed kernel yet");
    DeviceGuard g(h->device);
    const uint32_t n = std::min(h->tcount, kTimeSlots);
    const uint32_t last = (h->tcount - 1) % kTimeSlots;
    HIPCHK(h, hipEventSynchronize(h->tev[2 * last + 1]));
    double sum = 0.0;
    for (uint32_t i = 0; i < n; ++i) {
        const uint32_t slot = (h->tcount - 1 - i) % kTimeSlots;
        float one = 0.0f;
        HIPCHK(h, hipEventElapsedTime(&one, h->tev[2 * slot], h->tev[2 * slot + 1]));
        sum += one;
    }
    *ms = (float)(sum / n);
    return NETKV_OK;
}

netkv_status netkv_tier_counts(netkv_handle h, const netkv_requests_t *req, const int32_t *sel, uint64_t *counts,
                               void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    netkv_status st = check_requests(h, req);
    if (st) return st;
    if (!counts || (req->n_req && !sel)) return fail(h, NETKV_EINVAL, "sel and counts must not be NULL");
    if (!h->have_snap) return fail(h, NETKV_ENOTREADY, "no snapshot loaded");
    DeviceGuard g(h->device);
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(fill_u64_kernel, dim3(1), dim3(64), 0, s, counts, (uint64_t)5, 0ull);
    if (req->n_req)
        hipLaunchKernelGGL(tier_count_kernel, dim3((req->n_req + 255) / 256), dim3(256), 0, s, make_snap(h),
                           make_reqs(req), sel, (unsigned long long *)counts, h->errword);
    HIPCHK(h, hipGetLastError());
    return NETKV_OK;
}

netkv_status netkv_select_sequential(netkv_handle h, const netkv_requests_t *req, uint32_t cap, int32_t *out_idx,
                                     float *out_score, void *stream) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    netkv_status st = check_requests(h, req);
    if (st) return st;
    if (req->n_req && (!out_idx || !out_score)) return fail(h, NETKV_EINVAL, "out_idx and out_score must not be NULL");
    if (cap > 65535) return fail(h, NETKV_EINVAL, "cap must be <= 65535");
    if ((st = ready(h))) return st;
    if (req->n_req == 0) return NETKV_OK;
    DeviceGuard g(h->device);
    hipStream_t s = (hipStream_t)stream;
    const uint64_t R = req->n_req, P = h->P;
    if ((st = ensure_seq(h, R, P, true, false))) return st;
    const float *ll = nullptr;
    // validation (invalid requests get -1 / NaN), every request's scoring
    // record by batch index and the leaders' prefix lengths, by the batch
    // selection's ordering
    {
        TimingOff off(h);  // only the sequential kernel is timed
        const PairOut po{nullptr, nullptr, nullptr};
        // (with a row of its own per request the chains read a new row at every
        // step: on 48 decodes and 16 prefills 4,000 requests take 233 us so and
        // 252 from the batch order, 16,384 788 and 706, 65,536 2,893 and 2,366)
        if (R <= 512 * P && direct_batch(h, R, req->n_hashes, kDirectRecordTasks)) {
            // (the chain orders its requests with the selection's sort buffers)
            if ((st = ensure_scratch(h, h->sc, R, 0, req->n_hashes, s)) || (st = ensure_hotr(h, R)) ||
                (st = ensure_dlam(h, R)))
                return st;
            if ((st = run_direct(h, req, 1, out_idx, out_score, s, false, h->sc.hotr, h->dlam))) return st;
            ll = h->dlam;
        } else {
            if ((st = select_owned(h, req, 1, out_idx, out_score, po, false, 0xFFFFFFFFu, s, false, true, false)))
                return st;
            ll = h->sc.lead_lam;
        }
    }
    // requests grouped by prefill instance, batch order kept inside a group
    const Reqs rq = make_reqs(req);
    const uint32_t pbits = bits_for(P);
    const bool own_sort = R > kSortMinN && R <= kSortMaxN && h->sc.sort_cnt;
    hipLaunchKernelGGL(prefill_key_kernel, dim3((uint32_t)((R + 255) / 256)), dim3(256), 0, s, rq, (uint32_t)P,
                       (const Hot *)h->sc.hotr, h->seq_keys, own_sort ? nullptr : h->seq_vals);
    size_t tb = h->sc.sort_tmp_bytes;
    if (own_sort && pbits <= kSortMaxBits)   // one pass
        HIPCHK(h, sort_pass<false>(h, h->sc, h->seq_keys, nullptr, h->seq_keys_out, h->seq_perm, (uint32_t)R, 0, pbits,
                                   nullptr, nullptr, nullptr, nullptr, 0, 0, nullptr, nullptr, nullptr, s));
    else if (own_sort)
        HIPCHK(h, batch_sort_pairs(h, h->sc, h->seq_keys, nullptr, h->seq_keys_out, h->seq_perm, (uint32_t)R, pbits,
                                   s));
    else
        HIPCHK(h, rocprim::radix_sort_pairs<SortConfig>(h->sc.sort_tmp, tb, h->seq_keys, h->seq_keys_out,
                                                        h->seq_vals, h->seq_perm, (uint32_t)R, 0, pbits, s));
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(P, 256)), dim3(256), 0, s, h->seq_start, P, 0u);
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(P, 256)), dim3(256), 0, s, h->seq_end, P, 0u);
    hipLaunchKernelGGL(segment_kernel, dim3((uint32_t)((R + 255) / 256)), dim3(256), 0, s,
                       (const uint32_t *)h->seq_keys_out, (uint32_t)R, (uint32_t)P, h->seq_start, h->seq_end);
    HIPCHK(h, hipGetLastError());
    HIPCHK(h, time_begin(h, s));
    const Snap sn = make_snap(h);
    const Table t = make_table(h);
    const Hot *hr = h->sc.hotr;
    const uint32_t *ord = h->seq_perm, *b0 = h->seq_start, *b1 = h->seq_end;
    // one workgroup per prefill instance, all of them resident at once on
    // 256 CUs up to 1,024 prefills (256 threads: four workgroups per CU
    // within the register budget); a thread holds MAXC decodes
#define NETKV_SEQ(TT, MC)                                                                                       \
    hipLaunchKernelGGL((sequential_cached_kernel<TT, MC>), dim3((uint32_t)P), dim3(TT), 0, s, sn, t, rq, cap, hr, ll, \
                       ord, b0, b1, out_idx, out_score)
    const uint32_t Dn = h->D;
    if (Dn <= 64) NETKV_SEQ(64, 1);
    else if (Dn <= 256) NETKV_SEQ(256, 1);
    else if (Dn <= 512) NETKV_SEQ(256, 2);
    else if (Dn <= 1024) NETKV_SEQ(256, 4);
    else if (Dn <= 1536) NETKV_SEQ(256, 6);
    else if (Dn <= 2048) NETKV_SEQ(256, 8);
    else if (Dn <= 3072) NETKV_SEQ(256, 12);
    else if (Dn <= 4096) NETKV_SEQ(256, 16);
    else
        hipLaunchKernelGGL(sequential_kernel, dim3((uint32_t)P), dim3(kSeqThreads), 0, s, sn, t, rq, cap, hr, ll, ord,
                           b0, b1, out_idx, out_score);
#undef NETKV_SEQ
    HIPCHK(h, hipGetLastError());
    HIPCHK(h, time_end(h, s));
    return NETKV_OK;
}

netkv_status netkv_set_option(netkv_handle h, int option, uint32_t value) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    switch (option) {
    case NETKV_OPT_RUN_LEN:
        if (value > (1u << 20)) return fail(h, NETKV_EINVAL, "run length must be <= 2^20");
        h->run_len_opt = value;
        return NETKV_OK;
    case NETKV_OPT_REUSE:
        h->reuse_opt = value ? 1u : 0u;
        return NETKV_OK;
    case NETKV_OPT_POLICY:
        if (value > 2) return fail(h, NETKV_EINVAL, "policy must be 0 (full), 1 (no congestion) or 2 (topology only)");
        h->policy_opt = value;
        return NETKV_OK;
    case NETKV_OPT_LEAD_CAP:
        h->lead_cap_opt = value;
        return NETKV_OK;
    case NETKV_OPT_FORM:
        if (value > 2) return fail(h, NETKV_EINVAL, "form must be 0 (automatic), 1 (ordering pipeline) or 2 (bounded)");
        h->form_opt = value;
        return NETKV_OK;
    case NETKV_OPT_COLS:
        if (value != 0 && value != 1 && value != 2 && value != 3 && value != 4 && value != 6)
            return fail(h, NETKV_EINVAL, "decodes per lane must be 0 (automatic), 1, 2, 3, 4 or 6");
        h->cols_opt = value;
        return NETKV_OK;
    default:
        return fail(h, NETKV_EINVAL, "unknown option %d", option);
    }
}

netkv_status netkv_last_form(netkv_handle h, uint32_t *form) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (!form) return fail(h, NETKV_EINVAL, "form must not be NULL");
    if (!h->last_form) return fail(h, NETKV_ENOTREADY, "no batch selected yet");
    *form = h->last_form;
    return NETKV_OK;
}

netkv_status netkv_cache_info(netkv_handle h, uint64_t *index_slots, uint64_t *distinct_hashes,
                              uint64_t *shared_hashes, uint64_t *index_bytes) {
    if (!h) return NETKV_EINVAL;
    h->err.clear();
    if (!h->have_cache) return fail(h, NETKV_ENOTREADY, "no cache loaded (netkv_cache_load)");
    if (index_slots) *index_slots = 2 * h->buckets;
    if (distinct_hashes) *distinct_hashes = h->distinct;
    if (shared_hashes) *shared_hashes = h->rows - 1;
    if (index_bytes) *index_bytes = h->table_bytes;
    return NETKV_OK;
}

}  // extern "C"

// rc_cohort.hip -- batched ready-cohort control transition for AMD Instinct
// MI355X (gfx950): hand-written HIP kernels and the C ABI of rc_cohort.h.
//
// Kernels
//   rc_prep_kernel    once per handle: builds the route-table image that every
//                     workgroup stages into LDS.
//   rc_lanes_kernel   once per handle: what every plan lane needs to know of
//                     its session and cohort.
//   rc_chain_kernel, rc_table_kernel
//                     device-resident chain (Section 7 "Device resident"),
//                     with the full or the table image: one launch runs T
//                     chained steps; state lives in VGPRs, decisions never
//                     leave the chip.
//   rc_decide_kernel  host-round-trip step, part 1 (Section 7 "Host round
//                     trip"): decide + compact, publish a 4-byte word.
//   rc_body_kernel    host-round-trip step, part 2: the route body the host
//                     selected, or both in one launch, over the stepped
//                     sessions in order; effects at the slots that part 1
//                     left for them.
//
// Data layout (HBM, structure of arrays, leading dimension ld): state
// [W][ld], outcome [ld], effects [T][ld] for sid and tool, [T][ld][4] for the
// payload, n_taken [T][C].  A wavefront's lanes read the consecutive
// sessions of each of its cohorts from one word row (at most a few
// contiguous segments per row); an effect's payload is one 16-byte store.
//
// Launch plan (built on the host at create time).  Cohorts of at most 64
// sessions are packed, in order, into "sub-wavefront" bins that never need a
// workgroup barrier -- each into the first wavefront of the open bin with room
// for it, so a wavefront can hold several cohorts that are not neighbours --
// and larger cohorts go, in order, into "multi-wavefront" bins.  A bin is one
// workgroup of 4 wavefronts of plan lanes.  A cohort of at most 64 sessions never
// straddles a wavefront; a larger one starts on a wavefront boundary and spans
// whole wavefronts; no cohort straddles a bin.  Each wavefront has a 64-byte
// descriptor, from which rc_lanes_kernel makes a 12-byte record per lane.  The compaction
// (stable partition, taken first) is a wavefront ballot + mbcnt rank; a
// cohort spanning wavefronts adds an LDS exchange of per-wavefront popcounts
// behind one workgroup barrier per chunk of steps.
//
// Route-table image in LDS.
//   full:  row r < R holds the W masks table[r][w mod 16] * (w + 1); row R is
//          zero.  No arithmetic is left for the masks.
//   table: (when the full image would not fit) row r holds table[r][0..15],
//          row R is zero; the masks are formed in registers with full-rate
//          shifts and adds: the mask of w + 16 is the mask of w plus
//          table[r][w mod 16] << 4 (exact modulo 2^32).
// Ahead of the rows comes what the word-0 chain reads: word 0's masks (table
// image: with the tools and the rows' addresses), the route thresholds and,
// in CDF mode, a guide table: guide[b] is the route of outcome b * 2^(32-g),
// so the route of o lies in [guide[o >> (32-g)], guide[(o >> (32-g)) + 1]]
// (the indexed-search guide table of Chen and Asau, 1974); a binary search
// narrows it to three thresholds where a bucket holds more, and those are
// read together and counted.
//
// Per-word update, branch-free.  With d the decision and r the route:
//   sh = d ? 0 : (31 - r) mod 32      rotl by (r+1) mod 32 == rotr by sh
//   M  = masks of row (d ? r : R)      (zero when not taken)
//   oo = d ? 0 : o
//   S' = (rotr(S, sh) ^ M) + oo       one v_alignbit_b32 + one v_xad_u32

#include <hip/hip_runtime.h>

#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "rc_cohort.h"
#include "rc_plan.h"



namespace {

using namespace rc_plan;

// ---------------------------------------------------------------------------
// Device helpers
// ---------------------------------------------------------------------------

// MurmurHash3's 32-bit finalizer.
__device__ __forceinline__ uint32_t dev_fmix32(uint32_t h) {
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

__device__ __forceinline__ uint32_t rotr32(uint32_t x, uint32_t s) {
    return __builtin_amdgcn_alignbit(x, x, s);  // uses s mod 32
}

// Hide a value's provenance from the optimizer so that the branch-free
// update stays one alignbit + one xad per word (otherwise the select that
// made `sh`/`oo` is pushed into every word).
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
    asm("" : "+v"(v));
    return v;
}

// t * K for K = 1..16 from full-rate shifts and adds.  Every intermediate
// passes through opaque(), so the optimizer cannot re-fuse the chain into a
// quarter-rate v_mul_lo_u32.
template <int K>
__device__ __forceinline__ uint32_t mul_small(uint32_t t) {
    static_assert(K >= 1 && K <= 16, "K");
    if constexpr (K == 1) return opaque(t);
    else if constexpr (K == 2 || K == 4 || K == 8 || K == 16) {
        constexpr int s = K == 2 ? 1 : K == 4 ? 2 : K == 8 ? 3 : 4;
        return opaque(t << s);
    } else if constexpr (K == 3) return opaque((t << 1) + t);
    else if constexpr (K == 5) return opaque((t << 2) + t);
    else if constexpr (K == 9) return opaque((t << 3) + t);
    else if constexpr (K == 6) return opaque(mul_small<3>(t) << 1);
    else if constexpr (K == 7) return opaque((mul_small<3>(t) << 1) + t);
    else if constexpr (K == 10) return opaque(mul_small<5>(t) << 1);
    else if constexpr (K == 11) return opaque((mul_small<5>(t) << 1) + t);
    else if constexpr (K == 12) return opaque(mul_small<3>(t) << 2);
    else if constexpr (K == 13) return opaque((mul_small<3>(t) << 2) + t);
    else if constexpr (K == 14) return opaque(mul_small<7>(t) << 1);
    else return opaque((mul_small<7>(t) << 1) + t);  // 15
}

// (t << 4) + m in one instruction.
__device__ __forceinline__ uint32_t lshl4_add(uint32_t t, uint32_t m) {
    uint32_t r;
    asm("v_lshl_add_u32 %0, %1, 4, %2" : "=v"(r) : "v"(t), "v"(m));
    return r;
}

// A uniform value (kept in an SGPR) whose provenance is hidden.  Volatile,
// so that address arithmetic derived from it is not hoisted out of the loop
// it sits in, nor shared between two places that recompute it.
__device__ __forceinline__ uint32_t opaque_s(uint32_t v) {
    asm volatile("" : "+s"(v));
    return v;
}

__device__ __forceinline__ uint32_t lane_rank(uint64_t m) {
    // number of set bits of m below this lane
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint32_t uni(uint32_t v) {
    return __builtin_amdgcn_readfirstlane(v);
}

// Global accesses as a uniform base plus a 32-bit byte offset, so that they
// compile to the scalar-base + 32-bit vector-offset form.
__device__ __forceinline__ uint32_t ld32(const uint32_t* base, uint32_t byte_off) {
    return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(base) + byte_off);
}
// NT: nontemporal (streaming) store, for data the launch never reads again.
// It raises the write bandwidth of fully written cache lines; lines that
// several wavefronts fill piecewise are better left to the normal path.
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
template <bool NT = false>
__device__ __forceinline__ void st32(uint32_t* base, uint32_t byte_off, uint32_t v) {
    uint32_t* p = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(base) + byte_off);
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}
template <bool NT = false>
__device__ __forceinline__ void st128(uint32_t* base, uint32_t byte_off, uint4 v) {
    u32x4v* p = reinterpret_cast<u32x4v*>(reinterpret_cast<char*>(base) + byte_off);
    const u32x4v x = {v.x, v.y, v.z, v.w};
    if constexpr (NT) __builtin_nontemporal_store(x, p);
    else *p = x;
}

// A row base held in scalar registers, in the global address space (an opaque
// generic pointer would make the access a flat one).
typedef __attribute__((address_space(1))) uint32_t* gptr;
__device__ __forceinline__ uint32_t ldg(gptr base, uint32_t byte_off) {
    typedef const __attribute__((address_space(1))) char* bytes;
    return *reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(reinterpret_cast<bytes>(base) + byte_off);
}
__device__ __forceinline__ void stg_nt(gptr base, uint32_t byte_off, uint32_t v) {
    typedef __attribute__((address_space(1))) char* bytes;
    __builtin_nontemporal_store(v, reinterpret_cast<gptr>(reinterpret_cast<bytes>(base) + byte_off));
}

struct RouteArgs {
    uint32_t mode;        // RC_ROUTE_MOD / RC_ROUTE_CDF
    uint32_t n_routes;    // R
    uint32_t pow2_mask;   // R - 1 when R is a power of two, else 0
    uint32_t mod_recip;   // floor(2^32 / R) when R is not
    uint32_t is_pow2;
    uint32_t cdf_n;       // R - 1 thresholds
    uint32_t guide_shift; // 32 - g (CDF mode)
    uint32_t guide_top;   // largest step of the search inside a guide bucket
};

// o mod R by the reciprocal m = floor(2^32 / R): o m / 2^32 is below o / R by
// less than o / 2^32 < 1, so its floor is the quotient or one less, and one
// conditional subtraction finishes it (a general 32-bit remainder is about
// four times the instructions, on the serial path of the chain).  R = 23, us
// per launch with the remainder and with this: 100,000 sessions, W = 32, T =
// 16, 13.96 and 13.65; one 256-session cohort, W = 16, T = 32, 10.46 and
// 10.15; a million sessions, bound by HBM, the same.
__device__ __forceinline__ uint32_t mod_routes(uint32_t o, const RouteArgs& ra) {
    const uint32_t x = o - __umulhi(o, ra.mod_recip) * ra.n_routes;  // < 2 R
    const uint32_t y = x - ra.n_routes;
    return x < y ? x : y;  // y wraps above x when x < R
}

// Route kinds, fixed per kernel instantiation.
enum : int { RK_POW2 = 0, RK_MOD = 1, RK_CDF = 2 };

// Words of padding (2^32 - 1) behind the thresholds in LDS.
constexpr uint32_t CDF_PAD = 3;

// Route key: o mod R, or (CDF) from the LDS thresholds and guide table (see
// the file comment), with a branch-free search of fixed trip count.
template <int RK>
__device__ __forceinline__ uint32_t route_of(uint32_t o, const RouteArgs& ra,
                                             const uint32_t* cdf, const uint32_t* guide) {
    if constexpr (RK == RK_POW2) {
        return o & ra.pow2_mask;
    } else if constexpr (RK == RK_MOD) {
        return mod_routes(o, ra);
    } else {
        const uint32_t bkt = o >> ra.guide_shift;
        uint32_t pos = guide[bkt];
        if (ra.guide_top > 2u) {  // more than three thresholds in some bucket
            const uint32_t hi = guide[bkt + 1u];
            for (uint32_t stp = ra.guide_top; stp > 2u; stp >>= 1) {
                const uint32_t i = pos + stp;
                const uint32_t j = i < hi ? i : hi;              // min(i, hi)
                const uint32_t v = cdf[(j > 1u ? j : 1u) - 1u];  // always in range
                // both tests evaluated (no short circuit), so the read needs
                // no branch around it
                pos = ((i <= hi) & (v <= o)) ? i : pos;
            }
        }
        // At most three thresholds are left (one, where no bucket holds more):
        // read together, one LDS latency, and counted.  Those past the answer
        // are above o; the padding behind the last one counts only for
        // o = 2^32 - 1, whose route is R - 1.  Against a search to the end,
        // us per launch: routes of Zipf(3) over 23, one 256-session cohort, W
        // = 16, T = 32, 15.58 and 14.39; over 1,000, 100,000 sessions, W = 64,
        // T = 16, 35.17 and 34.08.  Even or Zipf(1.1) routes, at most one
        // threshold a bucket or few: within 1.5% either way.
        uint32_t below = cdf[pos] <= o;
        if (ra.guide_top > 1u) {
            const uint32_t v1 = cdf[pos + 1u], v2 = cdf[pos + 2u];
            below += (uint32_t)(v1 <= o) + (uint32_t)(v2 <= o);
        }
        pos += below;
        return pos < ra.cdf_n ? pos : ra.cdf_n;
    }
}

// Per-lane view of the plan for one bin.
struct LaneCohort {
    uint32_t s;       // session
    uint32_t c;       // cohort
    uint32_t b;       // first session of the cohort
    uint32_t k;       // cohort size
    uint64_t seg;     // lanes of the cohort inside this wavefront (sub-wave)
    uint32_t flags;
    bool active;
};

__device__ __forceinline__ LaneCohort lane_cohort(const uint32_t* __restrict__ wd,
                                                  const uint32_t* __restrict__ offsets, uint32_t lane) {
    LaneCohort L;
    const uint32_t s0 = uni(wd[WD_S0]);
    const uint32_t n_act = uni(wd[WD_NACT]);
    const uint32_t c_first = uni(wd[WD_CFIRST]);
    const uint32_t n_coh = uni(wd[WD_NCOH]);
    uint32_t b = uni(wd[WD_BFIRST]);
    uint32_t k = uni(wd[WD_KFIRST]);
    L.flags = uni(wd[WD_FLAGS]);
    L.s = s0 + lane;
    L.c = c_first;
    uint32_t lo = 0u;  // first lane of this lane's cohort
    if (n_coh > 1u) {
        // several sub-wavefront cohorts, listed in lane order: this lane's
        // is the last one that starts at or before it
        uint32_t at = 0u;
        for (uint32_t q = 0; q < n_coh; ++q) {
            const uint32_t cq = uni(wd[WD_LIST + q]);
            const uint32_t bq = offsets[cq];  // uniform addresses
            const uint32_t kq = offsets[cq + 1u] - bq;
            const bool mine = lane >= at;
            L.c = mine ? cq : L.c;
            b = mine ? bq : b;
            k = mine ? kq : k;
            lo = mine ? at : lo;
            at += kq;
        }
        L.s = b + (lane - lo);
    }
    L.b = b;
    L.k = k;
    L.active = lane < n_act;
    L.seg = 0;
    if (!(L.flags & WF_MULTI)) {
        uint32_t hi = lo + k;
        lo = lo < 64u ? lo : 64u;
        hi = hi < 64u ? hi : 64u;
        const uint64_t below_hi = hi >= 64u ? ~0ull : ((1ull << hi) - 1ull);
        const uint64_t below_lo = lo >= 64u ? ~0ull : ((1ull << lo) - 1ull);
        L.seg = below_hi & ~below_lo;
    }
    return L;
}

// Per lane of the plan, built once per handle: the session (TS_IDLE: no
// session), and what the compaction needs of its cohort.
constexpr uint32_t TS_IDLE = 0xFFFFFFFFu;
enum : uint32_t {
    TI_INC = 0,      // bits 0..7: index of the session in its cohort
    TI_SIZE = 8,     // bits 8..16: cohort size
    TI_LO = 17,      // bits 17..22: first lane of the cohort (sub-wavefront cohorts)
    TI_MULTI = 23,   // bit 23: the wavefront is part of a cohort of > 64 sessions, and of it:
    TI_WI = 24,      // bits 24..25: this wavefront's index in the cohort
    TI_NW = 26,      // bits 26..27: wavefronts of the cohort, minus one
    TI_FIRST = 28    // bits 28..29: first wavefront in the workgroup
};

// Also clears the handle's `n_words` counter words (a memset is 8 us of the
// host's time, this launch 3).
__global__ __launch_bounds__(256) void rc_lanes_kernel(const uint32_t* wdesc, const uint32_t* offsets,
                                                       uint32_t* lane_s, uint2* lane_i, uint32_t* words,
                                                       uint32_t n_words) {
    if (blockIdx.x == 0u && threadIdx.x < n_words) words[threadIdx.x] = 0u;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = blockIdx.x * 4u + (threadIdx.x >> 6);
    const LaneCohort L = lane_cohort(wdesc + (size_t)wave * WD_WORDS, offsets, lane);
    uint32_t v = 0u;
    if (L.flags & WF_MULTI)
        v = (1u << TI_MULTI) | (((L.flags >> 8) & 3u) << TI_WI) | ((((L.flags >> 16) - 1u) & 3u) << TI_NW) |
            (((L.flags >> 24) & 3u) << TI_FIRST);
    if (L.active) {
        const uint32_t in_c = L.s - L.b;
        v |= in_c | (L.k << TI_SIZE);
        if (!(L.flags & WF_MULTI)) v |= (lane - in_c) << TI_LO;
    }
    lane_s[(size_t)wave * 64u + lane] = L.active ? L.s : TS_IDLE;
    lane_i[(size_t)wave * 64u + lane] = make_uint2(L.active ? L.c : 0u, v);
}

// A lane's view of the plan from its record: the same fields as lane_cohort,
// without walking the wavefront's cohorts (scalar loads that wait for one
// another: a wavefront of eight small cohorts spent 1.2 us on them).
__device__ __forceinline__ LaneCohort lane_record(const uint32_t* __restrict__ lane_s,
                                                  const uint2* __restrict__ lane_i, size_t at, uint32_t s_lo,
                                                  uint32_t s_n) {
    const uint32_t s = lane_s[at];
    const uint2 i = lane_i[at];
    LaneCohort L;
    L.s = s;
    L.c = i.x;
    L.b = s - (i.y & 255u);
    L.k = (i.y >> TI_SIZE) & 511u;
    const uint32_t fl = uni(i.y);  // the same in every lane of the wavefront
    const uint32_t wi = (fl >> TI_WI) & 3u, nw = ((fl >> TI_NW) & 3u) + 1u, first = (fl >> TI_FIRST) & 3u;
    const bool multi = (fl >> TI_MULTI) & 1u;
    L.flags = multi ? (uint32_t)WF_MULTI | (wi << 8) | (nw << 16) | (first << 24) : 0u;
    L.active = s - s_lo < s_n;  // TS_IDLE is past every session
    const uint32_t lo = (i.y >> TI_LO) & 63u, hi = lo + L.k;
    L.seg = multi ? 0ull : (hi >= 64u ? ~0ull : ((1ull << hi) - 1ull)) & ~((1ull << lo) - 1ull);
    return L;
}

// The same from the wavefront's descriptor, for a wavefront of a cohort of
// more than 64 sessions: one scalar load.
__device__ __forceinline__ LaneCohort lane_descriptor(const uint32_t* __restrict__ wd, uint32_t lane, uint32_t s_lo,
                                                      uint32_t s_n) {
    LaneCohort L;
    L.s = uni(wd[WD_S0]) + lane;
    L.c = uni(wd[WD_CFIRST]);
    L.b = uni(wd[WD_BFIRST]);
    L.k = uni(wd[WD_KFIRST]);
    L.flags = uni(wd[WD_FLAGS]);
    L.active = lane < uni(wd[WD_NACT]) && L.s - s_lo < s_n;
    L.seg = 0ull;
    return L;
}

// A sub-wavefront bin's: the descriptor where one cohort has the whole
// wavefront, else the record.
__device__ __forceinline__ LaneCohort lane_view(const uint32_t* __restrict__ wd, const uint32_t* __restrict__ lane_s,
                                                const uint2* __restrict__ lane_i, size_t at, uint32_t lane,
                                                uint32_t s_lo, uint32_t s_n) {
    if (uni(wd[WD_NCOH]) > 1u) return lane_record(lane_s, lane_i, at, s_lo, s_n);
    LaneCohort L = lane_descriptor(wd, lane, s_lo, s_n);
    L.seg = L.k >= 64u ? ~0ull : ((1ull << L.k) - 1ull);  // the cohort starts at lane 0
    return L;
}

// ---------------------------------------------------------------------------
// Table image (built once per handle)
// ---------------------------------------------------------------------------
struct ImageArgs {
    const uint32_t* raw;  // [R][16]
    const uint32_t* cdf;  // [R-1]
    uint32_t* img;
    uint32_t* max_span;   // out: largest guide bucket span
    uint32_t n_routes, row_words, full, tab_words, tools_off, cdf_off, cdf_n;
    uint32_t guide_off, guide_n, guide_shift, total_words;
    uint32_t m0_words, rows_off;  // word-0 masks (full) or route pairs (table) at 0, rows at rows_off
};

// number of thresholds <= x (plain binary search over global memory)
__device__ __forceinline__ uint32_t count_le(const uint32_t* cdf, uint32_t n, uint32_t x) {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2u;
        if (cdf[mid] <= x) lo = mid + 1u; else hi = mid;
    }
    return lo;
}

// Table image: where row r's block 0 lies, in 16-byte units of LDS, as the
// high half of a control word.  Block q of row r is stored at block
// q ^ (r / 4 mod 4) of its 64 bytes (rows_off is a multiple of 16 words), so
// that lanes reading one block of random rows spread over all 16 bank groups
// (64-byte rows alone reach four) and every block is one XOR away.
__host__ __device__ __forceinline__ uint32_t table_row_field(uint32_t rows_off, uint32_t r) {
    return (rows_off / 4u + r * 4u + ((r >> 2) & 3u)) << 16;
}

__global__ __launch_bounds__(256) void rc_prep_kernel(ImageArgs a) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= a.total_words) return;
    const uint32_t R = a.n_routes;
    uint32_t v = 0;
    if (a.full && i < a.m0_words) {
        // word 0's taken mask of route i (row R and the padding: zero)
        if (i < R) v = a.raw[i * 16u];
    } else if (!a.full && i < a.m0_words) {
        // route pairs: word 0's taken mask, and the taken tool with the LDS
        // address of the route's row, as the control word holds them
        const uint32_t r = i >> 1;
        if (r < R) v = (i & 1u) ? ((a.raw[r * 16u + 1u] & 7u) << 6) | table_row_field(a.rows_off, r) : a.raw[r * 16u];
    } else if (i >= a.rows_off && i < a.rows_off + a.tab_words) {
        const uint32_t j = i - a.rows_off;
        if (a.full) {
            // row r: W masks, then one zero block of padding
            const uint32_t WM = a.row_words, RS = WM + 4u;
            const uint32_t r = j / RS, w = j % RS;
            if (r < R && w < WM) v = a.raw[r * 16u + (w & 15u)] * (w + 1u);
        } else {
            const uint32_t r = j / 16u, p = j % 16u;
            const uint32_t q = (p >> 2) ^ ((r >> 2) & 3u);
            const uint32_t w = 4u * q + (p & 3u);
            if (r < R) v = a.raw[r * 16u + w];
        }
    } else if (a.full && i >= a.tools_off && i < a.tools_off + R) {
        const uint32_t r = i - a.tools_off;
        v = (a.raw[r * 16u] & 7u) | ((a.raw[r * 16u + 1u] & 7u) << 8);
    } else if (i >= a.cdf_off && i < a.cdf_off + a.cdf_n + CDF_PAD) {
        v = i - a.cdf_off < a.cdf_n ? a.cdf[i - a.cdf_off] : 0xFFFFFFFFu;
    } else if (a.guide_n && i >= a.guide_off && i < a.guide_off + a.guide_n) {
        const uint32_t bkt = i - a.guide_off;
        const uint32_t last = a.guide_n - 1u;
        v = bkt == last ? a.cdf_n : count_le(a.cdf, a.cdf_n, bkt << a.guide_shift);
        if (bkt < last) {
            const uint32_t nxt = bkt + 1u == last ? a.cdf_n
                                                  : count_le(a.cdf, a.cdf_n, (bkt + 1u) << a.guide_shift);
            atomicMax(a.max_span, nxt - v);
        }
    }
    a.img[i] = v;
}

// ---------------------------------------------------------------------------
// Device-resident chain
// ---------------------------------------------------------------------------
struct ChainArgs {
    uint32_t* state;
    uint32_t* outcome;
    uint32_t* eff_sid;
    uint32_t* eff_tool;
    uint32_t* eff_payload;
    uint32_t* n_taken;
    const uint32_t* img;      // LDS image, img_words words
    const uint32_t* wdesc;    // [bins][waves][WD_WORDS]
    const uint32_t* lane_s;   // [bins][256] (see rc_lanes_kernel)
    const uint2* lane_i;
    RouteArgs ra;
    uint32_t ld, n_words, n_cohorts, thr, step0, n_steps;
    uint32_t s_lo, s_n;       // sessions of the stepped cohorts: [s_lo, s_lo + s_n)
    uint32_t bins_a_lo, bins_a_n, bins_b_lo, bins_b_n;  // sub-wave / multi-wave bins
    uint32_t img_words, tools_off, cdf_off, guide_off;  // in words
    uint32_t rows_off;     // full image: first word of the mask rows
    uint32_t chain_words;  // full image: words [0, chain_words) are what the word-0 chain reads
    const uint32_t* dbits;  // no-decision floor: [T][dwords] decision bitmap
    uint32_t dwords;
};

// No-decision floor: the bitmap word holding session s's decision at chained
// step t (bit s mod 32).  Idle lanes read session 0's word.
__device__ __forceinline__ uint32_t dword_of(const ChainArgs& a, uint32_t t, uint32_t s) {
    return a.dbits[(size_t)t * a.dwords + (s >> 5)];
}

// Workgroup barrier for LDS traffic only: each wavefront waits for its own
// LDS accesses (lgkmcnt 0; vmcnt and expcnt left at their maxima), not for
// its global loads and stores, which no other wavefront reads -- so state
// loads stay in flight across it.  (A workgroup release fence would wait for
// every outstanding global access as well.)
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_s_waitcnt(0xC07F);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Wait until at most N vector-memory accesses of this wavefront are
// outstanding (lgkmcnt and expcnt unconstrained).  They complete in issue
// order, so this waits for everything issued before the last N.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N <= 63, "vmcnt is a 6-bit count");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Full-image chain, split by what each word depends on.  A session's route,
// decision and next outcome at every step are functions of word 0 and the
// outcome alone; every other word only follows the per-step (mask row,
// rotation, addend) those choose.  Each chunk of up to TC steps runs as:
//   chain:   word 0 alone through the chunk -- two hashes, the route and the
//            decision per step -- recording (rotation | d << 5 | r << 6) and
//            the addend of every step; no store;
//   counts:  each wavefront publishes its taken count of every step of the
//            chunk (cohorts spanning wavefronts), then one barrier;
//   replay:  step by step, the words from the recorded control (one 16-byte
//            LDS read and two VALU ops per four words), the stable-partition
//            slot, and the effect stores.
// SPLIT: two lanes per session.  Wavefronts [0, NWAVE) ("A") run the plan's
// sessions: the chain, words [0, WA), the slots and the effects.
// Wavefronts [NWAVE, 2 NWAVE) ("B") mirror them lane for lane and replay
// words [WA, W) from the control the A lanes leave in LDS before the chunk's
// barrier; a second barrier closes the chunk when another follows.  The two
// roles run separate straight-line sequences with the same barriers.
// Rows of the mask image are W + 4 words apart (one zero block of padding
// shifts consecutive rows across the LDS banks), so block q of a row is an
// immediate offset from the row's byte offset.
// PIPED (W <= 32, WMAX = 16 or 32): three lanes per session; the A lanes
// keep only the chain and run it one 4-step chunk ahead, the B lanes replay
// words [0, 8) and emit the effects, the C lanes replay the rest (see PIPE
// below).
// FLOOR: the no-decision floor -- the A lanes read every decision from the
// bitmap instead of computing it (SPLIT: the first two chunks' words issued
// with the staging loads, later chunks' a chunk ahead).
template <int WMAX, bool EXACT, int NWAVE, int RK, bool MULTI, bool SPLIT, bool FLOOR, bool PIPED>
struct ChainF {
    static constexpr uint32_t CNT_STRIDE = NWAVE + 4;
    // Words per lane.  SPLIT: an A lane holds words [0, WA) of its session
    // and emits the effects; its B lane holds words [WA, WMAX).  At
    // WMAX = 32 the A lanes hold only the four payload words: once a
    // wavefront has issued stores, waiting for any earlier load means
    // waiting for everything on the vector-memory counter, so a lane that
    // emits effects should have no load left to wait for -- and the 28 words
    // of the B lanes then arrive while the effects go out.
    // PIPE (PIPED at WMAX = 16 or 32): three lanes per session.  The A
    // lanes hold only word 0 and the outcome and run the chain one 4-step
    // chunk ahead, storing nothing but the final outcome; behind it, the B
    // lanes replay each chunk over words [0, WP1) and emit the effects, and
    // the C lanes replay it over words [WP1, WMAX).  The chain of chunk
    // k + 1 then overlaps the replay of chunk k, where the two-role split
    // runs its 16-step chunks' chains and replays in turn; splitting the
    // replay over two roles gives it eight wavefronts per cohort to hide its
    // LDS and dependence latency.  The replay starts after one 4-step chunk,
    // so its state loads are not hidden behind a 16-step chain: with more
    // than one workgroup per CU and a one-operation route (mod R) the
    // two-role split is faster (the host decides).
    static constexpr bool PIPE = SPLIT && (WMAX == 32 || WMAX == 16) && PIPED;
    static constexpr int WP1 = 8;  // PIPE: words of the B lanes (the C lanes hold the rest)
    static constexpr int NROLE = PIPE ? 3 : SPLIT ? 2 : 1;
    static constexpr int WA = PIPE ? 0 : SPLIT ? (WMAX == 32 ? 4 : WMAX / 2) : WMAX;
    static constexpr int WB = SPLIT ? WMAX - WA : 0;
    static constexpr int WS = PIPE ? WMAX - WP1 : (WA > WB ? WA : WB);  // state registers per lane
    static constexpr int NBA = WA / 4, NBB = WB / 4;  // 16-byte blocks per lane
    static constexpr uint32_t RS = (WMAX + 4) * 4;       // row stride in bytes
    // steps per chunk (PIPE: two chunks in flight, each in its own half of
    // the 16-step control and count areas)
    static constexpr int TC = PIPE ? 4 : WMAX <= 32 ? 16 : 8;
    static constexpr uint32_t WG = NROLE * NWAVE * 64;
    static constexpr int SB = WMAX <= 32 ? (SPLIT ? 5 : 10) : (SPLIT ? 3 : 6);
    static constexpr uint32_t NLA = NWAVE * 64;  // lanes of the plan's sessions (the A lanes)
    // Bins of sub-wavefront cohorts (each cohort inside one wavefront) pass
    // their effects through an LDS stage: the lane of a session writes its
    // effect at the stage position of the lane that holds the session
    // numbered like the effect's slot, and reads back the effect whose slot
    // is its own session index -- one wavefront, so LDS order is all the
    // synchronization needed.  A wavefront's stores then cover its
    // sessions' contiguous slots, whole cache lines, and go out
    // nontemporal.  Cohorts spanning wavefronts store each effect directly
    // at its slot (an LDS exchange across wavefronts at every step costs
    // more than it saves).

    static __device__ __forceinline__ uint4 lds128(const uint32_t* lds, uint32_t byte_off) {
        return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(lds) + byte_off);
    }

    static __device__ __forceinline__ void run(const ChainArgs& a, uint32_t bin, uint4* lds4) {
        uint32_t* lds = reinterpret_cast<uint32_t*>(lds4);
        const uint32_t tid = threadIdx.x;
        const uint32_t lane = tid & 63u;
        const uint32_t wv = uni(tid >> 6);
        // 0: A; 1: B; 2 (PIPE): C -- uniform per wavefront
        const uint32_t role = SPLIT ? uni(wv / (uint32_t)NWAVE) : 0u;
        const bool role_b = role != 0u;
        const uint32_t wa = wv - role * (uint32_t)NWAVE;      // the plan wavefront it serves
        const uint32_t alane = wa * 64u + lane;                // lane index among the A lanes
        const uint32_t wbase = PIPE ? (role == 2u ? (uint32_t)WP1 : 0u) : (role_b ? (uint32_t)WA : 0u);  // first word
        const uint32_t W = a.n_words;
        const uint32_t R = a.ra.n_routes;
        const uint32_t T = a.n_steps;
        // The host reserves 16 steps of each: counts [16][NWAVE + 4], then
        // (SPLIT) the control handed to the replaying lanes -- addends
        // [16][NLA] and control words [16][NLA] -- then the effect stage of
        // sub-wavefront bins.  PIPE uses the first 2 TC steps of the count and
        // control areas (two chunks in flight).
        static_assert(TC <= 16 && (!PIPE || 2 * TC <= 16), "LDS control and count areas hold 16 steps");
        uint32_t* lds_cnt = lds + a.img_words;
        uint32_t* lds_add = lds_cnt + 16 * CNT_STRIDE;
        uint32_t* lds_ctl = lds_add + (SPLIT ? 16 * NLA : 0);
        uint32_t* stage_w = reinterpret_cast<uint32_t*>(lds_ctl + (SPLIT ? 16 * NLA : 0));
        uint4* stage_p = reinterpret_cast<uint4*>(stage_w + NLA);
        const uint32_t* lds_tools = lds + a.tools_off;

        const uint32_t rows_b = a.rows_off * 4u;  // byte offset of the mask rows in LDS
        LaneCohort L;
        // Cohorts of more than 64 sessions, from W = 9: the descriptor, which
        // spares the traffic of the records (12 bytes a session): 500,000
        // sessions in 256-session cohorts, W = 16, T = 1, 14.9 us against
        // 16.0 with the records; W = 32, T = 4, 30.0 and 31.2.  At W <= 8 the
        // records are no slower: W = 8, 130-session cohorts, within 1%.
        // Sub-wavefront bins: the records, but in the two-role split the
        // descriptor of a wavefront that one cohort has to itself.  What that
        // look costs the pipelined split: 100,000 sessions, W = 32, R = 256
        // CDF, T = 1, 6.7 us against 6.3 with 64-session cohorts and 6.7
        // against 6.4 with 32-session ones.  In the two-role split at W = 64
        // it wins up to 4% where such wavefronts stream from HBM and loses 2
        // to 6% where a wavefront has many cohorts (500,000 sessions, R = 200,
        // T = 4: 53.6 us against 56.0 with 64-session cohorts, 307 against 299
        // with one-session ones).  At W = 32 without it the compiler places
        // the blocks of the kernel's other half otherwise: 391 cohorts of 256
        // sessions, mod 256, T = 16, take 14.27 us against 14.07, their
        // no-decision floor 14.92 against 14.52.
        if constexpr (!MULTI && SPLIT && !PIPE)
            L = lane_view(a.wdesc + ((size_t)bin * NWAVE + wa) * WD_WORDS, a.lane_s, a.lane_i, (size_t)bin * NLA + alane,
                          lane, a.s_lo, a.s_n);
        else if constexpr (MULTI && WMAX >= 16)
            L = lane_descriptor(a.wdesc + ((size_t)bin * NWAVE + wa) * WD_WORDS, lane, a.s_lo, a.s_n);
        else
            L = lane_record(a.lane_s, a.lane_i, (size_t)bin * NLA + alane, a.s_lo, a.s_n);
        const uint32_t soff = L.s << 2;
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const u32x4* src = reinterpret_cast<const u32x4*>(a.img);
        const uint32_t n4 = a.img_words / 4u;
        // Unconditional loads (idle lanes read session 0 and never store), so
        // that no branch splits the in-order load sequence.
        uint32_t S[WS];
        const uint32_t loff = L.active ? soff : 0u;
        const uint32_t ldw = opaque_s(a.ld);
        uint32_t o = 0u;
        // Word 0 of the chain (A lanes) in a variable of its own: it is
        // loaded with the outcome before the first barrier, apart from the
        // state words that follow it.
        uint32_t s0 = 0u;
        uint32_t db[TC];   // FLOOR: the decision words of the first chunk (A lanes)
        uint32_t db1[TC];  // FLOOR, SPLIT: those of the second chunk
#pragma unroll
        for (int i = 0; i < TC; ++i) db[i] = db1[i] = 0u;
#pragma unroll
        for (int w = 0; w < WS; ++w) S[w] = 0u;
        // FLOOR: a chunk's decisions packed into one register (bit i = step
        // t0 + i), so the words die as soon as they arrive
        auto pack = [&](const uint32_t (&w)[TC]) {
            uint32_t m = 0u;
#pragma unroll
            for (int i = 0; i < TC; ++i) m |= ((w[i] >> (L.s & 31u)) & 1u) << i;
            return L.active ? m : 0u;
        };
        uint32_t dm = 0u, dm1 = 0u;
        // FLOOR: decision words, issued before the state words so that the
        // chain waits only for them and word 0
        auto load_db = [&]() {
            if constexpr (FLOOR) {
#pragma unroll
                for (int i = 0; i < TC; ++i)
                    if ((uint32_t)i < T) db[i] = dword_of(a, (uint32_t)i, L.active ? L.s : 0u);
            }
        };

        // (a1, a2) Staging.  SPLIT, A wavefronts: only what the word-0 chain
        // reads -- the chain section of the image (word-0 masks, CDF
        // thresholds, guide table), the outcome and word 0 (FLOOR: and the
        // first two chunks' decision words) -- so that the chain starts
        // after the first barrier.  SPLIT, B wavefronts (idle
        // until the chunk's control is published): the mask rows and tool
        // pairs, with direct-to-LDS loads that stay in flight across the
        // first (bare) barrier; every B lane waits for its own before the
        // barrier that precedes the first read of the rows.
        typedef __attribute__((address_space(3))) void lds_void;
        auto stage_a = [&]() {
            const uint32_t c4 = a.chain_words / 4u;
            for (uint32_t blk = wa; blk * 64u < c4; blk += NWAVE) {
                const uint32_t j = blk * 64u + lane;
                if (j < c4)
                    __builtin_amdgcn_global_load_lds((const void*)(src + j), (lds_void*)(lds4 + blk * 64u), 16, 0, 0);
            }
            o = ld32(a.outcome, loff);
            s0 = ld32(a.state, loff);
            if constexpr (FLOOR) {
                // The decision words of the first two chunks go out right
                // behind them, so that their latency overlaps the staging.
                // Steps past the chain read its last step's word: exactly
                // 2 TC loads follow, and waiting until at most that many are
                // outstanding completes everything issued before them (loads
                // retire in order).  They are packed before any store.
                asm volatile("" ::: "memory");
                const uint32_t ls = L.active ? L.s : 0u;
#pragma unroll
                for (int i = 0; i < TC; ++i) db[i] = dword_of(a, (uint32_t)i < T ? (uint32_t)i : T - 1u, ls);
#pragma unroll
                for (int i = 0; i < TC; ++i)
                    db1[i] = dword_of(a, (uint32_t)(TC + i) < T ? (uint32_t)(TC + i) : T - 1u, ls);
                asm volatile("" ::: "memory");
                wait_vmcnt<2 * TC>();  // chain section in LDS, outcome and word 0 in VGPRs
            } else {
                __builtin_amdgcn_s_waitcnt(0);  // chain section in LDS, outcome and word 0 in VGPRs
            }
        };
        auto stage_b = [&]() {
            const uint32_t c4 = a.chain_words / 4u;
            // PIPE: the B and C wavefronts share the blocks
            const uint32_t b0 = PIPE ? (role - 1u) * (uint32_t)NWAVE + wa : wa;
            constexpr uint32_t BSTR = PIPE ? 2u * NWAVE : NWAVE;
            for (uint32_t blk = b0; c4 + blk * 64u < n4; blk += BSTR) {
                const uint32_t j = c4 + blk * 64u + lane;
                if (j < n4)
                    __builtin_amdgcn_global_load_lds((const void*)(src + j), (lds_void*)(lds4 + c4 + blk * 64u),
                                                     16, 0, 0);
            }
        };
        // This lane's NW words (unconditional for idle lanes, which read
        // session 0 and never store, so that no branch splits the loads).
        auto load_words = [&](auto nw_c) {
            constexpr int NW = decltype(nw_c)::value;
#pragma unroll
            for (int w = 0; w < NW; ++w)
                if (EXACT || wbase + (uint32_t)w < W) S[w] = ld32(a.state + (size_t)(wbase + w) * ldw, loff);
        };
        // One lane per session: the first batch of the image, then the
        // outcome and the state words.  Vector-memory loads complete in
        // order, so the image batch can be written to LDS while the state
        // loads are still in flight.
        auto stage_single = [&]() {
            u32x4* dst = reinterpret_cast<u32x4*>(lds4);
            u32x4 v[SB];
#pragma unroll
            for (int k = 0; k < SB; ++k) {
                const uint32_t j = tid + (uint32_t)k * WG;
                v[k] = src[j < n4 ? j : n4 - 1u];
            }
            o = ld32(a.outcome, loff);
            load_db();
            load_words(std::integral_constant<int, WS>{});
            // Blocks past the image end repeat its last block (same value,
            // same address), so the writes need no branch either.
#pragma unroll
            for (int k = 0; k < SB; ++k) {
                const uint32_t j = tid + (uint32_t)k * WG;
                dst[j < n4 ? j : n4 - 1u] = v[k];
            }
            for (uint32_t j = tid + (uint32_t)SB * WG; j < n4; j += WG) dst[j] = src[j];
            __syncthreads();
            if constexpr (FLOOR) dm = pack(db);
            s0 = S[0];
        };

        // per-wavefront constants of the compaction
        const uint32_t in_c = L.s - L.b;
        bool f[4] = {false, false, false, false}, g[4] = {false, false, false, false};
        if constexpr (MULTI) {
            const uint32_t wi = (L.flags >> 8) & 0xFFu;
            const uint32_t nw = (L.flags >> 16) & 0xFFu;
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                f[k] = k < wi;  // wavefronts of the cohort before this one
                g[k] = k < nw;  // wavefronts of the cohort
            }
        }

        uint32_t step = a.step0;
        uint32_t* p_sid = a.eff_sid;
        uint32_t* p_tool = a.eff_tool;
        uint32_t* p_pay = a.eff_payload;
        uint32_t* p_cnt = a.n_taken;

        // The chain of the chunk starting at step t0 (A lanes): records its
        // control and addends, then publishes the counts and (SPLIT) the
        // control.  Chunk 0's chain runs ahead of the chunk loop, so that no
        // wait for the state words still in flight is placed before it.
        uint32_t ctl[TC], add[TC];
        // PIPE: first step slot of the half of the control and count areas
        // that holds the chunk starting at t0 (chunks alternate halves)
        auto half_of = [&](uint32_t t0) -> uint32_t {
            return PIPE ? ((t0 / (uint32_t)TC) & 1u) * (uint32_t)TC : 0u;
        };
        auto chain_chunk = [&](uint32_t t0) {
            const uint32_t n = (T - t0) < (uint32_t)TC ? (T - t0) : (uint32_t)TC;
#pragma unroll
            for (int i = 0; i < TC; ++i) {
                ctl[i] = 0u;
                add[i] = 0u;
            }
            if (!role_b) {
                // The chain is a serial dependence through two hashes per
                // step; raised issue priority keeps it moving while other
                // wavefronts of the SIMD replay (throughput work that fills
                // the gaps).
                __builtin_amdgcn_s_setprio(3);
                if constexpr (FLOOR) {
                    if (SPLIT && t0 == (uint32_t)TC)
                        dm = dm1;  // packed before the first chunk
                    else if (t0 != 0u)
                        dm = pack(db);
                }
                // chain: word 0 only
                uint32_t r = route_of<RK>(o, a.ra, lds + a.cdf_off, lds + a.guide_off);
                uint32_t m0 = lds[r];  // taken mask of word 0 on route r (chain section)
                // Branch-free: the decision is a lane mask, and the taken and
                // not-taken forms of the update differ only in masked
                // operands (a select the compiler would otherwise turn into a
                // divergent branch on this latency-bound path).
                const uint32_t act = L.active ? 1u : 0u;
#pragma unroll
                for (int i = 0; i < TC; ++i) {
                    if ((uint32_t)i >= n) continue;
                    uint32_t dbit;
                    if constexpr (FLOOR)
                        dbit = (dm >> i) & 1u;
                    else
                        dbit = act & (uint32_t)((dev_fmix32(s0 ^ o ^ step) & 0xFFFFu) < a.thr);
                    const uint32_t dmsk = 0u - dbit;  // all ones when taken
                    const uint32_t sh = (31u - r) & 31u;
                    const uint32_t rot = sh & ~dmsk;  // rotation 0 when taken
                    const uint32_t oo = o & ~dmsk;
                    // the step's control word: the rotation (bits 0..4, also
                    // the shift operand of the rotate), the decision (bit 5),
                    // the route (bits 6..15, for the tool pair) and the LDS
                    // address of the mask row the update reads -- route r's
                    // when taken, the zero row R's when not -- in 16-byte units
                    // (bits 16..31), made here in the latency-bound chain so
                    // that every replaying lane reads its row with one shift
                    ctl[i] = rot | (dmsk & 32u) | (r << 6) |
                             (((rows_b + __umul24(dbit ? r : R, RS)) >> 4) << 16);
                    add[i] = oo;
                    s0 = (rotr32(s0, rot) ^ (m0 & dmsk)) + oo;
                    o = dev_fmix32(s0);
                    r = route_of<RK>(o, a.ra, lds + a.cdf_off, lds + a.guide_off);
                    m0 = lds[r];
                    step += 1u;
                }
                // FLOOR: the next chunk's decision words, in flight during
                // this chunk's replay (SPLIT: chunk 1's are already packed)
                if constexpr (FLOOR) {
                    if ((!SPLIT || t0 >= (uint32_t)TC) && t0 + (uint32_t)TC < T) {
#pragma unroll
                        for (int i = 0; i < TC; ++i)
                            db[i] = t0 + (uint32_t)(TC + i) < T ? dword_of(a, t0 + TC + i, L.active ? L.s : 0u) : 0u;
                    }
                }
                // counts of the chunk's steps: every lane writes the same
                // (uniform) value to the same address, so no lane mask
                const uint32_t par = half_of(t0);
                if constexpr (MULTI) {
#pragma unroll
                    for (int i = 0; i < TC; ++i)
                        lds_cnt[(par + i) * CNT_STRIDE + wa] = (uint32_t)__popcll(__ballot((ctl[i] >> 5) & 1u));
                }
                // the control for the B lanes
                if constexpr (SPLIT) {
#pragma unroll
                    for (int i = 0; i < TC; ++i) {
                        lds_ctl[(par + i) * NLA + alane] = ctl[i];
                        lds_add[(par + i) * NLA + alane] = add[i];
                    }
                }
                // The two-role split keeps the raised priority through the A
                // lanes' replay too: their effect stores then start ahead of
                // the B lanes' bulk update (measured: 100,000 sessions 18.1 ->
                // 16.9 us together with the nontemporal payloads).
                if constexpr (!SPLIT || PIPE) __builtin_amdgcn_s_setprio(0);
            }
        };

        // Replay of the chunk starting at t0 over this lane's 16-byte word
        // blocks [QLO, QHI), with (EFF: the A lanes, or the B lanes under
        // PIPE) the slots and effects, step by step.  PREF: the LDS reads of
        // step i + 1 (mask blocks and, with EFF, the tool pair) are issued
        // before step i is computed; past the chunk's last step they
        // read the zero row (valid addresses, values unused).  The step count
        // is re-read so that no per-step condition stays live across the
        // phases.
        const uint32_t my = alane;  // this lane's stage position
        auto replay = [&](uint32_t t0, auto qlo_c, auto qhi_c, auto eff_c, auto pref_c) {
            constexpr int QLO = decltype(qlo_c)::value;
            constexpr int QHI = decltype(qhi_c)::value;
            constexpr int NQ = QHI - QLO;
            constexpr bool EFF = decltype(eff_c)::value;
            constexpr bool PREF = decltype(pref_c)::value;
            const uint32_t n = (T - t0) < (uint32_t)TC ? (T - t0) : (uint32_t)TC;
            const uint32_t nr = opaque_s(n);
            const uint32_t* cq0 = lds_cnt + (L.flags >> 24) + half_of(t0) * CNT_STRIDE;
            const uint32_t qoff = (wbase + 4u * QLO) * 4u;  // byte offset of the first block in a row
            // Cohorts spanning wavefronts: the chunk's counts are all in LDS
            // before its replay starts, so each wavefront combines them once
            // per chunk, lane-parallel -- lane i holds step i's taken count
            // of the cohort (n1v) and of its wavefronts before this one
            // (prev) -- and each step takes its two values with a readlane
            // (lanes past the chunk read valid count slots, unused).
            uint32_t n1v = 0u, prev = 0u;
            if constexpr (EFF && MULTI) {
                const uint32_t* q = cq0 + (lane < (uint32_t)TC ? lane : 0u) * CNT_STRIDE;
                const uint32_t c0 = q[0], c1 = q[1], c2 = q[2], c3 = q[3];
                n1v = (g[0] ? c0 : 0u) + (g[1] ? c1 : 0u) + (g[2] ? c2 : 0u) + (g[3] ? c3 : 0u);
                prev = (f[0] ? c0 : 0u) + (f[1] ? c1 : 0u) + (f[2] ? c2 : 0u);
            }
            uint4 mc[NQ];
            uint32_t tpc = 0u;
            if constexpr (PREF) {
                const uint32_t c = ctl[0];
                const uint32_t rowoff = ((c >> 16) << 4) + qoff;
#pragma unroll
                for (int q = 0; q < NQ; ++q) mc[q] = lds128(lds, rowoff + 16u * q);
                if constexpr (EFF) tpc = lds_tools[(c >> 6) & 0x3FFu];
            }
#pragma unroll
            for (int i = 0; i < TC; ++i) {
                uint4 mn[NQ];
                uint32_t tpn = 0u;
                if constexpr (!PREF) {
                    const uint32_t c = ctl[i];
                    const uint32_t rowoff = ((c >> 16) << 4) + qoff;
#pragma unroll
                    for (int q = 0; q < NQ; ++q) mc[q] = lds128(lds, rowoff + 16u * q);
                    if constexpr (EFF) tpc = lds_tools[(c >> 6) & 0x3FFu];
                }
                if (PREF && i + 1 < TC) {
                    const uint32_t c = ctl[i + 1];
                    const uint32_t rowoff = ((c >> 16) << 4) + qoff;
#pragma unroll
                    for (int q = 0; q < NQ; ++q) mn[q] = lds128(lds, rowoff + 16u * q);
                    if constexpr (EFF) tpn = lds_tools[(c >> 6) & 0x3FFu];
                }
                if ((uint32_t)i < nr) {
                    const uint32_t c = ctl[i];
                    const uint32_t oo = add[i];
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const int b = 4 * (QLO + q);
                        if (!EXACT && wbase + (uint32_t)b >= W) continue;
                        S[b] = (rotr32(S[b], c) ^ mc[q].x) + oo;
                        S[b + 1] = (rotr32(S[b + 1], c) ^ mc[q].y) + oo;
                        S[b + 2] = (rotr32(S[b + 2], c) ^ mc[q].z) + oo;
                        S[b + 3] = (rotr32(S[b + 3], c) ^ mc[q].w) + oo;
                    }
                    if constexpr (EFF) {
                        const bool dk = (c >> 5) & 1u;
                        const uint32_t tool = (tpc >> (dk ? 8u : 0u)) & 7u;

                        // (a5) stable partition, taken first
                        const uint64_t bal = __ballot(dk);
                        uint32_t n1, rank_t;
                        if constexpr (MULTI) {
                            n1 = __builtin_amdgcn_readlane(n1v, i);
                            rank_t = __builtin_amdgcn_readlane(prev, i) + lane_rank(bal);
                        } else {
                            const uint64_t bs = bal & L.seg;
                            n1 = (uint32_t)__popcll(bs);
                            rank_t = lane_rank(bs);
                        }
                        const uint32_t slot = L.b + (dk ? rank_t : n1 + (in_c - rank_t));

                        // (a7) emit; slot - b < k always holds (the test keeps
                        // a compaction defect from becoming a write outside
                        // the cohort)
                        const bool put = L.active && slot - L.b < L.k;
                        if constexpr (MULTI) {
                            // a wavefront's taken and not-taken sessions land
                            // in two contiguous slot runs, so its 16-byte
                            // payloads fill most lines whole: those go out
                            // nontemporal; the 4-byte fields, spread over more
                            // partly filled lines, through the L2
                            if (put) {
                                st32(p_sid, slot << 2, L.s);
                                st32(p_tool, slot << 2, tool);
                                st128<true>(p_pay, slot << 4, make_uint4(S[0], S[1], S[2], S[3]));
                                if (in_c == 0u) st32(p_cnt, L.c << 2, n1);
                            }
                        } else {
                            // a cohort's sessions sit in consecutive lanes,
                            // so session `slot` is held at stage position
                            // my + (slot - s); sid < 2^28 leaves room for
                            // the tool
                            if (put) {
                                const uint32_t pos = my + (slot - L.s);
                                stage_w[pos] = L.s | (tool << 28);
                                stage_p[pos] = make_uint4(S[0], S[1], S[2], S[3]);
                            }
                            asm volatile("" ::: "memory");
                            if (L.active) {
                                const uint32_t w = stage_w[my];
                                const uint4 pv = stage_p[my];
                                st32<true>(p_sid, soff, w & 0x0FFFFFFFu);
                                st32<true>(p_tool, soff, w >> 28);
                                st128<true>(p_pay, soff << 2, pv);
                                if (in_c == 0u) st32(p_cnt, L.c << 2, n1);
                            }
                            asm volatile("" ::: "memory");  // this step's reads before the next step's writes
                        }
                        p_sid += ldw;
                        p_tool += ldw;
                        p_pay += 4u * ldw;
                        p_cnt += a.n_cohorts;
                    }
                }
                if (PREF && i + 1 < TC) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q) mc[q] = mn[q];
                    if constexpr (EFF) tpc = tpn;
                }
            }
        };

        // (a9) store this lane's NW words and (A lanes) the next outcome (the
        // row addresses are recomputed from a fresh copy of ld rather than
        // kept live across the chain)
        auto store_state = [&](auto nw_c, bool with_outcome) {
            constexpr int NW = decltype(nw_c)::value;
            if (L.active) {
                const uint32_t ld_st = opaque_s(a.ld);
#pragma unroll
                for (int w = 0; w < NW; ++w)
                    if (EXACT || wbase + (uint32_t)w < W) st32<true>(a.state + (size_t)(wbase + w) * ld_st, soff, S[w]);
                if (with_outcome) st32<true>(a.outcome, soff, o);
            }
        };
        auto bare_barrier = []() {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        using Z = std::integral_constant<int, 0>;
        using NA = std::integral_constant<int, NBA>;
        using NB = std::integral_constant<int, NBB>;
        using Yes = std::integral_constant<bool, true>;
        using No = std::integral_constant<bool, false>;
        // the B lanes of a 28-word split read each step's masks when the step
        // starts (no room for a second set of mask registers)
        using PrefB = std::integral_constant<bool, (NBB <= 4)>;

        // Each role runs its own straight-line sequence to the end, with the
        // same barriers per chunk, so that the compiler's wait analysis sees
        // one role's accesses at a time.  Chunk 0 runs outside the chunk
        // loop: the compiler flushes every outstanding vector-memory access
        // in the preheader of a loop that stores without loading.
        if constexpr (PIPE) {
            // The same barriers in both roles: a bare one after staging, then
            // one per chunk.  Barrier k + 1 publishes chunk k's control and
            // counts (A) and closes the replay of chunk k - 1 (B); chunk k + 2
            // reuses chunk k's half only after barrier k + 2, when its replay
            // is done.
            if (!role_b) {
                stage_a();
                bare_barrier();
                if constexpr (FLOOR) {
                    dm = pack(db);
                    dm1 = pack(db1);
                }
                for (uint32_t t0 = 0; t0 < T; t0 += TC) {
                    chain_chunk(t0);
                    lds_barrier();
                }
                if (L.active) st32<true>(a.outcome, soff, o);
            } else {
                stage_b();
                bare_barrier();
                auto read_ctl = [&](uint32_t t0) {
                    const uint32_t par = half_of(t0);
#pragma unroll
                    for (int i = 0; i < TC; ++i) {
                        ctl[i] = lds_ctl[(par + i) * NLA + alane];
                        add[i] = lds_add[(par + i) * NLA + alane];
                    }
                };
                // B (words [0, WP1), effects) and C (the rest): the same
                // barriers, each with its own straight-line sequence
                auto replay_role = [&](auto nw_c, auto nq_c, auto eff_c) {
                    constexpr int NWR = decltype(nw_c)::value;
                    load_words(nw_c);
                    // the row loads issued before the NWR state loads have
                    // landed (with W < WMAX fewer were issued: wait for all)
                    wait_vmcnt<EXACT ? NWR : 0>();
                    lds_barrier();
                    read_ctl(0u);
                    wait_vmcnt<0>();  // every word is needed at the first step
                    replay(0u, Z{}, nq_c, eff_c, No{});
                    for (uint32_t t0 = TC; t0 < T; t0 += TC) {
                        lds_barrier();
                        read_ctl(t0);
                        replay(t0, Z{}, nq_c, eff_c, No{});
                    }
                    store_state(nw_c, false);
                };
                if (role == 1u)
                    replay_role(std::integral_constant<int, WP1>{}, std::integral_constant<int, WP1 / 4>{}, Yes{});
                else
                    replay_role(std::integral_constant<int, WMAX - WP1>{},
                                std::integral_constant<int, (WMAX - WP1) / 4>{}, No{});
            }
        } else if constexpr (SPLIT) {
            if (!role_b) {
                stage_a();
                bare_barrier();
                // FLOOR: the decision words of the first two chunks (issued in
                // stage_a) are packed before any store is issued: once stores
                // are outstanding, waiting for a load drains them too.
                load_words(std::integral_constant<int, WA>{});
                if constexpr (FLOOR) {
                    dm = pack(db);
                    dm1 = pack(db1);
                }
                chain_chunk(0u);
                lds_barrier();  // publishes chunk 0's counts and control
                // The replay needs all WA words at its first step; an explicit
                // wait here (nothing else is outstanding) keeps the compiler
                // from repeating it, step after step, behind the effect stores.
                wait_vmcnt<0>();
                replay(0u, Z{}, NA{}, Yes{}, Yes{});
                for (uint32_t t0 = TC; t0 < T; t0 += TC) {
                    lds_barrier();  // every wavefront is done with the previous chunk's
                    chain_chunk(t0);
                    lds_barrier();
                    replay(t0, Z{}, NA{}, Yes{}, Yes{});
                }
                store_state(std::integral_constant<int, WA>{}, true);
            } else {
                stage_b();
                bare_barrier();
                load_words(std::integral_constant<int, WB>{});
                // the row loads issued before the WB state loads have landed
                // (with W < WMAX fewer state loads were issued: wait for all)
                wait_vmcnt<EXACT ? WB : 0>();
                lds_barrier();
                auto read_ctl = [&]() {
#pragma unroll
                    for (int i = 0; i < TC; ++i) {
                        ctl[i] = lds_ctl[i * NLA + alane];
                        add[i] = lds_add[i * NLA + alane];
                    }
                };
                read_ctl();
                wait_vmcnt<0>();  // every word is needed at the first step
                replay(0u, Z{}, NB{}, No{}, PrefB{});
                for (uint32_t t0 = TC; t0 < T; t0 += TC) {
                    lds_barrier();
                    lds_barrier();
                    read_ctl();
                    replay(t0, Z{}, NB{}, No{}, PrefB{});
                }
                store_state(std::integral_constant<int, WB>{}, false);
            }
        } else {
            stage_single();
            chain_chunk(0u);
            if constexpr (MULTI) lds_barrier();
            replay(0u, Z{}, NA{}, Yes{}, Yes{});
            for (uint32_t t0 = TC; t0 < T; t0 += TC) {
                if constexpr (MULTI) lds_barrier();
                chain_chunk(t0);
                if constexpr (MULTI) lds_barrier();
                replay(t0, Z{}, NA{}, Yes{}, Yes{});
            }
            store_state(std::integral_constant<int, WMAX>{}, true);
        }
    }
};

// One workgroup per bin: blocks [0, bins_a_n) take the sub-wavefront bins,
// the rest the multi-wavefront bins.  The two-role chain at W = 32 runs two
// 512-lane workgroups per CU, so it is held to four wavefronts per SIMD (at
// most 128 VGPRs); the pipelined split (W = 16 or 32) runs two 768-lane
// workgroups per CU, six wavefronts per SIMD (at most 80 VGPRs).  At W = 64
// the two-role chain needs more registers and runs one workgroup per CU.
template <int WMAX, bool EXACT, int NWAVE, int RK, bool FLOOR, bool PIPED>
__global__ __launch_bounds__((WMAX >= 32 || (PIPED && WMAX == 16) ? (PIPED && WMAX <= 32 ? 3 : 2) : 1) * NWAVE * 64,
                             WMAX == 32 ? (PIPED ? 6 : 4) : (PIPED && WMAX == 16 ? 6 : 1))
void rc_chain_kernel(ChainArgs a) {
    extern __shared__ uint4 lds4[];
    constexpr bool SPLIT = WMAX >= 32 || (PIPED && WMAX == 16);
    if (blockIdx.x < a.bins_a_n)
        ChainF<WMAX, EXACT, NWAVE, RK, false, SPLIT, FLOOR, PIPED>::run(a, a.bins_a_lo + blockIdx.x, lds4);
    else
        ChainF<WMAX, EXACT, NWAVE, RK, true, SPLIT, FLOOR, PIPED>::run(a, a.bins_b_lo + (blockIdx.x - a.bins_a_n), lds4);
}

// ---------------------------------------------------------------------------
// Device-resident chain, table image
// ---------------------------------------------------------------------------
struct TableArgs {
    uint32_t* state;
    uint32_t* outcome;
    uint32_t* eff_sid;
    uint32_t* eff_tool;
    uint32_t* eff_payload;
    uint32_t* n_taken;
    const uint32_t* img;      // LDS image: [route pairs | thresholds | guide] (chain_words), raw rows
    const uint32_t* lane_s;   // [bins][256]
    const uint2* lane_i;      // [bins][256]: cohort, TI_ fields
    RouteArgs ra;
    uint32_t ld, n_words, n_cohorts, thr, step0, n_steps;
    uint32_t s_lo, s_n;       // sessions of the stepped cohorts: [s_lo, s_lo + s_n)
    uint32_t bins_a_lo, bins_a_n, bins_b_lo, n_units;
    uint32_t img_words, chain_words, cdf_off, guide_off, zero_row;  // zero_row: row R's control field
    const uint32_t* dbits;    // no-decision floor: [T][dwords] decision bitmap
    uint32_t dwords;
};

// NB = ceil(W / 16) bands of 16 words.  The masks are table[r][w mod 16] *
// (w + 1): column j's masks over the bands are t * (j + 1), + (t << 4), ...
// with t = table[r][j], so the words are split over wavefronts by column and
// each reads only its columns of the row.
//
// A workgroup is four wavefronts of plan lanes (up to 256 sessions) in four
// roles, lane for lane, 16 wavefronts in all (one of each role per SIMD):
//   A  chains word 0 and the outcome, one 4-step chunk ahead, and leaves
//      every step's control (rotation, decision, tool, mask row) and addend
//      in LDS, with the taken counts of each wavefront;
//   B  replays columns 0..3 and emits the effects;
//   C, D  replay columns 4..9 and 10..15.
// One LDS barrier per chunk: barrier g publishes chunk g and closes the
// replay of chunk g - 1 (two chunks in flight, in alternating halves).
//
// Workgroups are persistent: the image is staged once and the workgroup
// takes every gridDim-th bin, its loads issued one bin ahead into registers,
// so that the loads and the final stores of a bin overlap the steps of its
// neighbours.  Only B emits effects, and B issues no load: loads and stores
// retire through one in-order counter, and a load behind a step's effects
// would wait for them.  A fetches B's words and plan lane with its own and
// hands them over in LDS.
//
// The form that this replaces ran one lane per session, all W words and the
// effects in it, eight wavefronts to a workgroup and a barrier per step: few
// sessions left most SIMDs idle, many waited together.  Measured, before and
// after, us per launch: 60,007 sessions in 467 cohorts, W = 48, R = 1000, T =
// 24: 38.2 -> 28.9; 5,000 sessions, W = 64, R = 1024 CDF, T = 40: 56.8 -> 26.9;
// one 100-session cohort, W = 33, T = 20: 31.0 -> 12.9; 130,000 sessions, W =
// 64, T = 16: 34.0 -> 28.7.  A million sessions, W = 64, R = 1024, T = 16: 212
// -> 205 (4.4 TB/s): bound by HBM with the loads, effects and final stores of
// a bin taking turns (203 with nearly all arithmetic removed); few sessions
// are bound by VALU issue (about 316 instructions per step and SIMD at W =
// 64, of them 3 per word).  Also measured on it: progress counters in LDS in
// place of the barriers 215 us (a wavefront's partly filled lines then meet
// their neighbours' later), single wavefronts walking bins on their own with
// one lane per session 232 us.
//
// Where it is slower than the form it replaces: one or two steps that stream
// from HBM (from about 300,000 sessions) in partly filled wavefronts, whose
// bins hold few sessions each.  A million sessions, T = 1, before and after:
// 33-session cohorts, W = 49, 77 -> 105; 130-session cohorts, W = 64, 99 ->
// 115; full wavefronts, W = 64, 84 -> 86.  It moves the same bytes there.
// Words fetched two units ahead made those launches 20% slower still, bins in
// XCD-contiguous order won 4% on them and lost 2% on full wavefronts, and one
// lane per session in 1,024-lane persistent workgroups was slower than both.
template <int NB, int RK, bool FLOOR>
struct ChainT {
    static constexpr int TC = 4;
    static constexpr uint32_t NW = 4, NL = NW * 64u;
    static constexpr uint32_t CNT = 8;  // words per step of the counts (cohorts read four from their first)

    // LDS after the image, in 16-byte units
    static constexpr uint32_t L_CNT = 2 * TC * CNT / 4, L_CTL = 2 * TC * NL / 2, L_HAND = 2 * (NB + 1) * NL,
                              L_STAGE = NL + NL / 4;
    static constexpr uint32_t LDS_AFTER = (L_CNT + L_CTL + L_HAND + L_STAGE) * 16u;

    // This lane's words of columns [J0, J0 + NC).  The row's base is walked in
    // scalar registers, hidden at every row: folded together, the sums become
    // 64-bit vector addresses.  A row past W repeats the last one read, so
    // that no load needs a branch (its value is unused).
    template <int J0, int NC>
    static __device__ __forceinline__ void load_cols(const TableArgs& a, uint32_t s, uint32_t (&S)[NB * NC]) {
        const uint32_t off = s << 2;
        const uint32_t ld = opaque_s(a.ld);
        gptr row = (gptr)(a.state + (size_t)J0 * ld);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                asm volatile("" : "+s"(row));
                S[b * NC + j] = ldg(row, off);
                const uint32_t w = 16 * b + J0 + j, next = j + 1 < NC ? w + 1 : w + 17 - NC;
                row += (b < NB - 1 && (b < NB - 2 || j + 1 < NC)) || next < a.n_words ? (size_t)(next - w) * ld : 0u;
            }
    }

    template <int J0, int NC>
    static __device__ __forceinline__ void store_cols(const TableArgs& a, uint32_t s, const uint32_t (&S)[NB * NC]) {
        const uint32_t off = s << 2;
        const uint32_t ld = opaque_s(a.ld);
        gptr row = (gptr)(a.state + (size_t)J0 * ld);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const uint32_t w = 16 * b + J0 + j, next = j + 1 < NC ? w + 1 : w + 17 - NC;
                asm volatile("" : "+s"(row));
                if (b < NB - 1 || w < a.n_words) stg_nt(row, off, S[b * NC + j]);
                row += (size_t)(next - w) * ld;
            }
    }

    // One step of columns [J0, J0 + NC): words past W (last band) start
    // anywhere, are never stored and feed nothing, so they need no branch.
    template <int J0, int NC>
    static __device__ __forceinline__ void update(uint32_t (&S)[NB * NC], const uint32_t (&t)[NC], uint32_t c,
                                                  uint32_t oo) {
        if constexpr (NC > 0) update_col<J0, NC, 0>(S, t, c, oo);
    }
    template <int J0, int NC, int J>
    static __device__ __forceinline__ void update_col(uint32_t (&S)[NB * NC], const uint32_t (&t)[NC], uint32_t c,
                                                      uint32_t oo) {
        if constexpr (J < NC) {
            uint32_t m = mul_small<J0 + J + 1>(t[J]);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                S[b * NC + J] = (rotr32(S[b * NC + J], c) ^ m) + oo;
                if (b + 1 < NB) m = lshl4_add(t[J], m);
            }
            update_col<J0, NC, J + 1>(S, t, c, oo);
        }
    }

    // Columns of the row a control word points at: 16-byte block q of a row
    // is one XOR away from its block 0 (see rc_prep_kernel).
    template <int J0, int NC>
    static __device__ __forceinline__ void row_cols(const uint32_t* lds, uint32_t ctl, uint32_t (&t)[NC]) {
        const uint32_t rb = ctl >> 12;
        const char* p = reinterpret_cast<const char*>(lds);
        if constexpr (J0 == 0) {
            const uint4 v = *reinterpret_cast<const uint4*>(p + rb);
            t[0] = v.x; t[1] = v.y; t[2] = v.z; t[3] = v.w;
        } else if constexpr (J0 == 4) {
            const uint4 v = *reinterpret_cast<const uint4*>(p + (rb ^ 16u));
            const uint2 u = *reinterpret_cast<const uint2*>(p + (rb ^ 32u));
            t[0] = v.x; t[1] = v.y; t[2] = v.z; t[3] = v.w; t[4] = u.x; t[5] = u.y;
        } else {
            const uint2 u = *reinterpret_cast<const uint2*>(p + (rb ^ 32u) + 8u);
            const uint4 v = *reinterpret_cast<const uint4*>(p + (rb ^ 48u));
            t[0] = u.x; t[1] = u.y; t[2] = v.x; t[3] = v.y; t[4] = v.z; t[5] = v.w;
        }
    }

    static __device__ __forceinline__ uint32_t bin_of(const TableArgs& a, uint32_t u) {
        return u < a.bins_a_n ? a.bins_a_lo + u : a.bins_b_lo + (u - a.bins_a_n);
    }
    // session of plan lane `al` of unit u, idle past the launch's units and
    // outside the stepped sessions
    static __device__ __forceinline__ uint32_t lane_session(const TableArgs& a, uint32_t u, uint32_t al) {
        return u < a.n_units ? a.lane_s[(size_t)bin_of(a, u) * NL + al] : TS_IDLE;
    }
    static __device__ __forceinline__ bool stepped(const TableArgs& a, uint32_t s) { return s - a.s_lo < a.s_n; }

    static __device__ __forceinline__ void run(const TableArgs& a, uint4* lds4) {
        uint32_t* lds = reinterpret_cast<uint32_t*>(lds4);
        const uint32_t tid = threadIdx.x;
        const uint32_t lane = tid & 63u;
        const uint32_t wv = uni(tid >> 6);
        const uint32_t role = wv >> 2, wa = wv & 3u;  // wavefronts go to SIMDs in turn: one of each role on each
        const uint32_t al = wa * 64u + lane;
        const uint32_t T = a.n_steps;
        const uint32_t G = gridDim.x, u0 = blockIdx.x;

        uint4* p = lds4 + a.img_words / 4u;
        uint32_t* cnt = reinterpret_cast<uint32_t*>(p);
        uint2* ctl = reinterpret_cast<uint2*>(p + L_CNT);
        uint4* hand = p + L_CNT + L_CTL;              // [2][NB + 1][NL]: B's words and plan lane
        uint4* stage_p = hand + L_HAND;
        uint32_t* stage_w = reinterpret_cast<uint32_t*>(stage_p + NL);

        typedef __attribute__((address_space(3))) void lds_void;
        const uint4* img = reinterpret_cast<const uint4*>(a.img);
        const uint32_t c4 = a.chain_words / 4u, n4 = a.img_words / 4u;
        // 16-byte blocks [lo, hi) of the image, by wavefronts w of nw
        auto stage = [&](uint32_t lo, uint32_t hi, uint32_t w, uint32_t nw) {
            for (uint32_t blk = lo + w * 64u; blk < hi; blk += nw * 64u)
                if (blk + lane < hi)
                    __builtin_amdgcn_global_load_lds((const void*)(img + blk + lane), (lds_void*)(lds4 + blk), 16, 0, 0);
        };
        auto bare_barrier = []() {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };

        if (role == 0u) {
            // -- A ----------------------------------------------------------
            stage(0u, c4, wa, NW);
            uint32_t sN = lane_session(a, u0, al), sNN = lane_session(a, u0 + G, al);
            uint32_t P[4 * NB], po;
            uint2 pi;
            uint32_t dN[TC];
#pragma unroll
            for (int i = 0; i < 4 * NB; ++i) P[i] = 0u;
            // words, outcome and plan lane of unit u
            auto fetch = [&](uint32_t u) {
                const uint32_t s = stepped(a, sN) ? sN : a.s_lo;
                po = ld32(a.outcome, s << 2);
                load_cols<0, 4>(a, s, P);
                pi = a.lane_i[(size_t)bin_of(a, u) * NL + al];
                if constexpr (FLOOR) {
#pragma unroll
                    for (int i = 0; i < TC; ++i)
                        dN[i] = a.dbits[(size_t)((uint32_t)i < T ? (uint32_t)i : T - 1u) * a.dwords + (s >> 5)];
                }
            };
            fetch(u0);
            wait_vmcnt<0>();  // chain section in LDS
            bare_barrier();
            __builtin_amdgcn_s_setprio(3);
            const uint2* pairs = reinterpret_cast<const uint2*>(lds);
            uint32_t half = 0u, hb = 0u;
            for (uint32_t u = u0; u < a.n_units; u += G, hb ^= 1u) {
                const bool act = stepped(a, sN);
                const uint32_t ss = act ? sN : a.s_lo;
                uint32_t s0 = P[0], o = po;
                uint4* h = hand + hb * (NB + 1) * NL + al;
#pragma unroll
                for (int b = 0; b < NB; ++b) h[b * NL] = make_uint4(P[4 * b], P[4 * b + 1], P[4 * b + 2], P[4 * b + 3]);
                h[NB * NL] = make_uint4(pi.x, pi.y, act ? sN : TS_IDLE, 0u);
                uint32_t dw[TC];
                if constexpr (FLOOR) {
#pragma unroll
                    for (int i = 0; i < TC; ++i) dw[i] = dN[i];
                }
                sN = sNN;
                if (u + G < a.n_units) {
                    fetch(u + G);
                    sNN = lane_session(a, u + 2u * G, al);
                }
                uint32_t step = a.step0;
                uint32_t r = route_of<RK>(o, a.ra, lds + a.cdf_off, lds + a.guide_off);
                uint2 pr = pairs[r];
                const uint32_t actb = act ? 1u : 0u;
                for (uint32_t t0 = 0; t0 < T; t0 += TC, half ^= 1u) {
                    const uint32_t n = T - t0;
                    uint32_t dnx[TC];
                    if constexpr (FLOOR) {
                        // the next chunk's decision words, in flight during this one
#pragma unroll
                        for (int i = 0; i < TC; ++i) {
                            const uint32_t t = t0 + TC + i;
                            dnx[i] = t0 + TC < T ? a.dbits[(size_t)(t < T ? t : T - 1u) * a.dwords + (ss >> 5)] : 0u;
                        }
                    }
#pragma unroll
                    for (int i = 0; i < TC; ++i) {
                        if ((uint32_t)i >= n) continue;
                        uint32_t dbit;
                        if constexpr (FLOOR)
                            dbit = actb & (dw[i] >> (ss & 31u));
                        else
                            dbit = actb & (uint32_t)((dev_fmix32(s0 ^ o ^ step) & 0xFFFFu) < a.thr);
                        const uint32_t dm = 0u - dbit;  // all ones when taken
                        const uint32_t rot = (31u - r) & 31u & ~dm;
                        const uint32_t oo = o & ~dm;
                        // control: rotation (bits 0..4), decision (5), tool
                        // (6..8), LDS address of the mask row / 16 (16..31)
                        const uint32_t nt = ((pr.x & 7u) << 6) | a.zero_row;
                        const uint32_t c = (dbit ? pr.y : nt) | rot | (dm & 32u);
                        ctl[(half * TC + i) * NL + al] = make_uint2(c, oo);
                        cnt[(half * TC + i) * CNT + wa] = (uint32_t)__popcll(__ballot(dbit != 0u));
                        s0 = (rotr32(s0, rot) ^ (pr.x & dm)) + oo;
                        o = dev_fmix32(s0);
                        r = route_of<RK>(o, a.ra, lds + a.cdf_off, lds + a.guide_off);
                        pr = pairs[r];
                        step += 1u;
                    }
                    if constexpr (FLOOR) {
#pragma unroll
                        for (int i = 0; i < TC; ++i) dw[i] = dnx[i];
                    }
                    lds_barrier();
                }
            }
        } else if (role == 1u) {
            // -- B ----------------------------------------------------------
            stage(c4, n4, wa, 3u * NW);
            bare_barrier();
            wait_vmcnt<0>();  // rows in LDS before the barrier that publishes the first chunk
            uint32_t half = 0u, hb = 0u;
            for (uint32_t u = u0; u < a.n_units; u += G, hb ^= 1u) {
                uint32_t S[4 * NB];
                uint32_t s = 0u, coh = 0u, inf = 0u;
                uint32_t* p_sid = a.eff_sid;
                uint32_t* p_tool = a.eff_tool;
                uint32_t* p_pay = a.eff_payload;
                uint32_t* p_cnt = a.n_taken;
                for (uint32_t t0 = 0; t0 < T; t0 += TC, half ^= 1u) {
                    lds_barrier();
                    if (t0 == 0u) {
                        const uint4* h = hand + hb * (NB + 1) * NL + al;
#pragma unroll
                        for (int b = 0; b < NB; ++b) {
                            const uint4 v = h[b * NL];
                            S[4 * b] = v.x; S[4 * b + 1] = v.y; S[4 * b + 2] = v.z; S[4 * b + 3] = v.w;
                        }
                        const uint4 v = h[NB * NL];
                        coh = v.x;
                        inf = v.y;
                        s = v.z;
                    }
                    const uint32_t fl = uni(inf);
                    const bool multi = (fl >> TI_MULTI) & 1u;
                    const bool act = s != TS_IDLE;
                    const uint32_t in_c = inf & 255u, k = (inf >> TI_SIZE) & 511u, b0 = s - in_c;
                    const uint32_t n = (T - t0) < (uint32_t)TC ? (T - t0) : (uint32_t)TC;
                    // the cohort's taken counts: lane i combines step i's
                    uint32_t n1v = 0u, prev = 0u;
                    if (multi) {
                        const uint32_t* q = cnt + (half * TC + (lane & 3u)) * CNT + ((fl >> TI_FIRST) & 3u);
                        const uint32_t wi = (fl >> TI_WI) & 3u, nw = ((fl >> TI_NW) & 3u) + 1u;
                        const uint32_t q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
                        n1v = q0 + q1 + (nw > 2u ? q2 : 0u) + (nw > 3u ? q3 : 0u);
                        prev = (wi > 0u ? q0 : 0u) + (wi > 1u ? q1 : 0u) + (wi > 2u ? q2 : 0u);
                    }
                    const uint32_t lo = (inf >> TI_LO) & 63u, hi = lo + k;  // this lane's cohort, if sub-wavefront
                    const uint64_t seg = multi ? ~0ull
                                               : (hi >= 64u ? ~0ull : ((1ull << hi) - 1ull)) & ~((1ull << lo) - 1ull);
                    // the chunk's control and mask columns, read together
                    // (steps past the last one repeat it)
                    uint2 cas[TC];
                    uint32_t ts[TC][4];
#pragma unroll
                    for (int i = 0; i < TC; ++i)
                        cas[i] = ctl[(half * TC + ((uint32_t)i < n ? (uint32_t)i : n - 1u)) * NL + al];
#pragma unroll
                    for (int i = 0; i < TC; ++i) row_cols<0, 4>(lds, cas[i].x, ts[i]);
#pragma unroll
                    for (int i = 0; i < TC; ++i) {
                        if ((uint32_t)i >= n) continue;
                        const uint2 ca = cas[i];
                        update<0, 4>(S, ts[i], ca.x, ca.y);
                        const bool dk = (ca.x >> 5) & 1u;
                        const uint32_t tool = (ca.x >> 6) & 7u;
                        // (a5) stable partition, taken first
                        const uint64_t bal = __ballot(dk);
                        const uint64_t bs = bal & seg;
                        uint32_t n1, rank_t = lane_rank(bs);
                        if (multi) {
                            n1 = __builtin_amdgcn_readlane(n1v, i);
                            rank_t += __builtin_amdgcn_readlane(prev, i);
                        } else {
                            n1 = (uint32_t)__popcll(bs);
                        }
                        const uint32_t in_slot = dk ? rank_t : n1 + (in_c - rank_t);
                        const uint32_t slot = b0 + in_slot;
                        // (a7) emit; in_slot < k always holds (the test keeps
                        // a compaction defect from becoming a write outside
                        // the cohort)
                        const bool put = act && in_slot < k;
                        if (multi) {
                            if (put) {
                                st32<true>(p_sid, slot << 2, s);
                                st32<true>(p_tool, slot << 2, tool);
                                st128<true>(p_pay, slot << 4, make_uint4(S[0], S[1], S[2], S[3]));
                                if (in_c == 0u) st32(p_cnt, coh << 2, n1);
                            }
                        } else {
                            // through the LDS stage of this wavefront, so
                            // that its stores cover contiguous slots
                            if (put) {
                                const uint32_t pos = al + (slot - s);
                                stage_w[pos] = s | (tool << 28);
                                stage_p[pos] = make_uint4(S[0], S[1], S[2], S[3]);
                            }
                            asm volatile("" ::: "memory");
                            if (act) {
                                const uint32_t w = stage_w[al];
                                const uint4 pv = stage_p[al];
                                st32<true>(p_sid, s << 2, w & 0x0FFFFFFFu);
                                st32<true>(p_tool, s << 2, w >> 28);
                                st128<true>(p_pay, s << 4, pv);
                                if (in_c == 0u) st32(p_cnt, coh << 2, n1);
                            }
                            asm volatile("" ::: "memory");  // this step's reads before the next step's writes
                        }
                        p_sid += a.ld;
                        p_tool += a.ld;
                        p_pay += 4u * a.ld;
                        p_cnt += a.n_cohorts;
                    }
                }
                // (a9) the words of this role and the next outcome
                if (s != TS_IDLE) {
                    store_cols<0, 4>(a, s, S);
                    st32<true>(a.outcome, s << 2, dev_fmix32(S[0]));
                }
            }
        } else {
            // -- C, D -------------------------------------------------------
            stage(c4, n4, wv - NW, 3u * NW);
            auto replay_role = [&](auto j0_c) {
                constexpr int J0 = decltype(j0_c)::value;
                constexpr int NC = 6;
                uint32_t sN = lane_session(a, u0, al), sNN = lane_session(a, u0 + G, al);
                uint32_t P[NB * NC];
#pragma unroll
                for (int i = 0; i < NB * NC; ++i) P[i] = 0u;
                load_cols<J0, NC>(a, stepped(a, sN) ? sN : a.s_lo, P);
                bare_barrier();
                wait_vmcnt<0>();  // rows in LDS before the barrier that publishes the first chunk
                uint32_t half = 0u;
                for (uint32_t u = u0; u < a.n_units; u += G) {
                    uint32_t S[NB * NC];
#pragma unroll
                    for (int i = 0; i < NB * NC; ++i) S[i] = P[i];
                    const uint32_t s = sN;
                    sN = sNN;
                    if (u + G < a.n_units) {
                        load_cols<J0, NC>(a, stepped(a, sN) ? sN : a.s_lo, P);
                        sNN = lane_session(a, u + 2u * G, al);
                    }
                    for (uint32_t t0 = 0; t0 < T; t0 += TC, half ^= 1u) {
                        const uint32_t n = (T - t0) < (uint32_t)TC ? (T - t0) : (uint32_t)TC;
                        lds_barrier();
                        uint2 cas[TC];
                        uint32_t ts[TC][NC];
#pragma unroll
                        for (int i = 0; i < TC; ++i)
                            cas[i] = ctl[(half * TC + ((uint32_t)i < n ? (uint32_t)i : n - 1u)) * NL + al];
#pragma unroll
                        for (int i = 0; i < TC; ++i) row_cols<J0, NC>(lds, cas[i].x, ts[i]);
#pragma unroll
                        for (int i = 0; i < TC; ++i) {
                            if ((uint32_t)i >= n) continue;
                            update<J0, NC>(S, ts[i], cas[i].x, cas[i].y);
                        }
                    }
                    // the loads of the next unit are long done: wait for them
                    // ahead of the stores, not behind
                    wait_vmcnt<0>();
                    if (stepped(a, s)) store_cols<J0, NC>(a, s, S);
                }
            };
            if (role == 2u)
                replay_role(std::integral_constant<int, 4>{});
            else
                replay_role(std::integral_constant<int, 10>{});
        }
    }
};

template <int NB, int RK, bool FLOOR>
__global__ __launch_bounds__(1024, 4) void rc_table_kernel(TableArgs a) {
    extern __shared__ uint4 lds4[];
    ChainT<NB, RK, FLOOR>::run(a, lds4);
}

// ---------------------------------------------------------------------------
// Host round trip
// ---------------------------------------------------------------------------

// Part 1: decide and compact one step.  Writes n_taken and, for every
// stepped session, where[s] = slot | d << 31 (its slot in the stable
// partition of its cohort), and adds the workgroup's taken count to
// ctr[parity] (the 4-byte word the host reads).  Block 0 clears the other
// parity's counter for the next step.  A workgroup takes up to four bins at
// a time, and there are at most DECIDE_WGS (see decide_few): the adds to the one word are
// performed one after the other, about 11 ns each (a workgroup and an add per
// bin: 391 bins spent 4.3 us of 6.5 on them).
struct DecideArgs {
    const uint32_t* state;
    const uint32_t* outcome;
    uint32_t* n_taken;
    uint32_t* where;          // session s of the stepped range at where[s - where_lo]
    uint32_t* ctr;            // [2]
    const uint32_t* lane_s;   // [bins][256] (see rc_lanes_kernel)
    const uint2* lane_i;
    uint32_t thr, step, t_index, n_cohorts;
    uint32_t s_n;             // stepped sessions, from where_lo
    uint32_t bins_a_lo, bins_a_n, bins_b_lo, n_units, parity, where_lo;
};

__global__ __launch_bounds__(1024) void rc_decide_kernel(DecideArgs a) {
    __shared__ uint32_t cnt[2][16 + 4];  // taken counts of the wavefronts (a cohort reads four from its first)
    __shared__ uint32_t wg_taken;
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wv = uni(tid >> 6);
    const uint32_t per = blockDim.x / 256u;  // bins at a time
    if (tid == 0u) {
        wg_taken = 0u;
        if (blockIdx.x == 0u) a.ctr[a.parity ^ 1u] = 0u;
    }
    uint32_t taken = 0u, buf = 0u;
    // the same trips for every wavefront: one barrier each
    for (uint32_t u0 = blockIdx.x * per; u0 < a.n_units; u0 += gridDim.x * per, buf ^= 1u) {
        const uint32_t u = u0 + (wv >> 2);
        LaneCohort L{};
        if (u < a.n_units) {
            const uint32_t bin = u < a.bins_a_n ? a.bins_a_lo + u : a.bins_b_lo + (u - a.bins_a_n);
            L = lane_record(a.lane_s, a.lane_i, (size_t)bin * 256u + (tid & 255u), a.where_lo, a.s_n);
        }
        uint32_t s0w = 0, o = 0;
        if (L.active) {
            s0w = ld32(a.state, L.s << 2);
            o = ld32(a.outcome, L.s << 2);
        }
        const bool dk = L.active && ((dev_fmix32(s0w ^ o ^ a.step) & 0xFFFFu) < a.thr);
        const uint64_t bal = __ballot(dk);
        if (lane == 0u) cnt[buf][wv] = (uint32_t)__popcll(bal);
        __syncthreads();
        uint32_t n1, rank_t;
        if (!(L.flags & WF_MULTI)) {
            const uint64_t bs = bal & L.seg;
            n1 = (uint32_t)__popcll(bs);
            rank_t = lane_rank(bs);
        } else {
            const uint32_t wi = (L.flags >> 8) & 0xFFu, nw = (L.flags >> 16) & 0xFFu;
            const uint32_t* q = &cnt[buf][(wv & ~3u) + (L.flags >> 24)];
            uint32_t before = 0;
            n1 = 0;
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                const uint32_t ci = uni(q[i]);
                n1 += (i < nw) ? ci : 0u;
                before += (i < wi) ? ci : 0u;
            }
            rank_t = before + lane_rank(bal);
        }
        if (L.active) {
            const uint32_t slot = L.b + (dk ? rank_t : n1 + ((L.s - L.b) - rank_t));
            if (L.s == L.b) a.n_taken[(size_t)a.t_index * a.n_cohorts + L.c] = n1;
            a.where[L.s - a.where_lo] = slot | (dk ? 0x80000000u : 0u);
        }
        taken += (uint32_t)__popcll(bal);
    }
    if (lane == 0u && taken) atomicAdd(&wg_taken, taken);
    __syncthreads();
    if (tid == 0u && wg_taken) atomicAdd(&a.ctr[a.parity], wg_taken);
}

// Part 2: the route body the host selected -- the taken one, the not-taken
// one, or both in one launch when the step has sessions of both kinds.  One
// lane per session, in session order: all state accesses are whole lines.
// (A launch per body, each over the slots of both kinds, read and wrote the
// lines that both kinds share twice: 100,000 sessions, W = 32, 7.4 + 6.8 us
// a step against 6.0 for both at once, and 11 us between them.)
struct BodyArgs {
    uint32_t* state;
    uint32_t* outcome;
    uint32_t* eff_sid;
    uint32_t* eff_tool;
    uint32_t* eff_payload;
    const uint32_t* where;  // session s at where[s - lo]
    const uint32_t* raw;    // [R][16]
    const uint32_t* cdf;    // thresholds and guide table of the handle's image
    const uint32_t* guide;
    RouteArgs ra;
    uint32_t ld, n_words, lo, hi, t_index;
};

enum : int { BODY_NOT = 0, BODY_TAKEN = 1, BODY_BOTH = 2 };

template <int WMAX, bool EXACT, int BODY>
__global__ __launch_bounds__(256) void rc_body_kernel(BodyArgs a) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= a.hi - a.lo) return;
    const uint32_t e = a.where[i];
    const bool dk = BODY == BODY_BOTH ? (e >> 31) != 0u : BODY == BODY_TAKEN;
    const uint32_t slot = e & 0x7FFFFFFFu;
    const uint32_t s = a.lo + i;
    // never by what the decide kernel wrote: another kind, or a slot outside
    // the stepped sessions
    if (dk != ((e >> 31) != 0u) || slot - a.lo >= a.hi - a.lo) return;
    const uint32_t W = a.n_words;
    const uint32_t soff = s << 2;
    const uint32_t o = ld32(a.outcome, soff);
    const uint32_t ld = opaque_s(a.ld);
    uint32_t S[WMAX];
#pragma unroll
    for (int w = 0; w < WMAX; w += 4) {
        if (!EXACT && (uint32_t)w >= W) {
            S[w] = S[w + 1] = S[w + 2] = S[w + 3] = 0u;
            continue;
        }
        // in the last block, words past W repeat the last one: no branch between the loads
#pragma unroll
        for (int q = w; q < w + 4; ++q)
            S[q] = ld32(a.state + (size_t)(EXACT || (uint32_t)q < W ? (uint32_t)q : W - 1u) * ld, soff);
    }
    const uint32_t r = a.ra.mode == RC_ROUTE_CDF ? route_of<RK_CDF>(o, a.ra, a.cdf, a.guide)
                     : a.ra.is_pow2 ? route_of<RK_POW2>(o, a.ra, a.cdf, a.guide)
                                    : route_of<RK_MOD>(o, a.ra, a.cdf, a.guide);
    const uint32_t* row = a.raw + r * 16u;
    const uint32_t tool = row[dk ? 1u : 0u] & 7u;
    if constexpr (BODY == BODY_NOT) {
        const uint32_t sh = (31u - r) & 31u;
#pragma unroll
        for (int w = 0; w < WMAX; ++w) S[w] = rotr32(S[w], sh) + o;
    } else {
        uint32_t m[WMAX < 16 ? WMAX : 16];
#pragma unroll
        for (int w = 0; w < (WMAX < 16 ? WMAX : 16); ++w) m[w] = 0u;
        if (dk) {
#pragma unroll
            for (int w = 0; w < (WMAX < 16 ? WMAX : 16); w += 4) {
                const uint4 v = *reinterpret_cast<const uint4*>(row + w);
                m[w] = v.x; m[w + 1] = v.y; m[w + 2] = v.z; m[w + 3] = v.w;
            }
        }
        const uint32_t sh = opaque(dk ? 0u : ((31u - r) & 31u));
        const uint32_t oo = opaque(dk ? 0u : o);
#pragma unroll
        for (int w = 0; w < WMAX; ++w) S[w] = (rotr32(S[w], sh) ^ (m[w & 15] * (uint32_t)(w + 1))) + oo;
    }
#pragma unroll
    for (int w = 0; w < WMAX; ++w)
        if (EXACT || (uint32_t)w < W) st32(a.state + (size_t)w * ld, soff, S[w]);
    const size_t slice = (size_t)a.t_index * a.ld;
    st32(a.eff_sid + slice, slot << 2, s);
    st32(a.eff_tool + slice, slot << 2, tool);
    st128(a.eff_payload + slice * 4u, slot << 4, make_uint4(S[0], S[1], S[2], S[3]));
    st32(a.outcome, soff, dev_fmix32(S[0]));
}

// Clears n words (a kernel rather than a memset, so that callers that
// capture the work into a graph record no memset node).
__global__ __launch_bounds__(64) void rc_clear_kernel(uint32_t* p, uint32_t n) {
    const uint32_t i = blockIdx.x * 64u + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Scratch of rc_cohort_run_chain_noalloc: two counter words, padding, then
// the slots of at most RC_NOALLOC_MAX_SESSIONS
// sessions.  Each device holds its own copy for the life of the process.
constexpr uint32_t NOALLOC_WHERE_OFF = 64u;
__device__ __align__(256) uint32_t rc_noalloc_scratch[NOALLOC_WHERE_OFF + RC_NOALLOC_MAX_SESSIONS];

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

typedef void (*ChainFn)(ChainArgs);
typedef void (*TableFn)(TableArgs);
typedef void (*BodyFn)(BodyArgs);

// The pipelined split exists for the full image at WMAX = 16 and 32.
bool has_piped(uint32_t wmax, bool full) { return full && (wmax == 32u || wmax == 16u); }

template <int WMAX, bool EXACT, int RK, bool FLOOR>
ChainFn chain_fn(bool piped) {
    if constexpr (WMAX == 32 || WMAX == 16)
        if (piped) return rc_chain_kernel<WMAX, EXACT, 4, RK, FLOOR, true>;
    return rc_chain_kernel<WMAX, EXACT, 4, RK, FLOOR, false>;
}

template <int WMAX, bool EXACT, bool FLOOR>
ChainFn chain_fn_rk(bool piped, int rk) {
    return rk == RK_POW2 ? chain_fn<WMAX, EXACT, RK_POW2, FLOOR>(piped)
         : rk == RK_MOD ? chain_fn<WMAX, EXACT, RK_MOD, FLOOR>(piped)
                        : chain_fn<WMAX, EXACT, RK_CDF, FLOOR>(piped);
}

template <bool FLOOR>
ChainFn pick_chain_t(uint32_t wmax, bool exact, bool piped, int rk) {
    switch (wmax) {
        case 4: return exact ? chain_fn_rk<4, true, FLOOR>(piped, rk) : chain_fn_rk<4, false, FLOOR>(piped, rk);
        case 8: return exact ? chain_fn_rk<8, true, FLOOR>(piped, rk) : chain_fn_rk<8, false, FLOOR>(piped, rk);
        case 16: return exact ? chain_fn_rk<16, true, FLOOR>(piped, rk) : chain_fn_rk<16, false, FLOOR>(piped, rk);
        case 32: return exact ? chain_fn_rk<32, true, FLOOR>(piped, rk) : chain_fn_rk<32, false, FLOOR>(piped, rk);
        default: return exact ? chain_fn_rk<64, true, FLOOR>(piped, rk) : chain_fn_rk<64, false, FLOOR>(piped, rk);
    }
}

ChainFn pick_chain(uint32_t wmax, bool exact, bool piped, int rk, bool floor) {
    return floor ? pick_chain_t<true>(wmax, exact, piped, rk) : pick_chain_t<false>(wmax, exact, piped, rk);
}

// Table image (W > 16): kernel of nb = ceil(W / 16) bands, and its LDS after
// the image.
template <int NB, bool FLOOR>
TableFn table_fn(int rk) {
    return rk == RK_POW2 ? rc_table_kernel<NB, RK_POW2, FLOOR>
         : rk == RK_MOD ? rc_table_kernel<NB, RK_MOD, FLOOR>
                        : rc_table_kernel<NB, RK_CDF, FLOOR>;
}

TableFn pick_table(uint32_t nb, int rk, bool floor) {
    switch (nb) {
        case 2: return floor ? table_fn<2, true>(rk) : table_fn<2, false>(rk);
        case 3: return floor ? table_fn<3, true>(rk) : table_fn<3, false>(rk);
        default: return floor ? table_fn<4, true>(rk) : table_fn<4, false>(rk);
    }
}

uint32_t table_lds_after(uint32_t nb) {
    return nb == 2u ? ChainT<2, 0, false>::LDS_AFTER : nb == 3u ? ChainT<3, 0, false>::LDS_AFTER
                                                                : ChainT<4, 0, false>::LDS_AFTER;
}

// The pipelined split for a launch: at most one workgroup per CU, or a
// chain whose route is a threshold search (CDF mode), whose longer step
// makes the overlap pay at any launch size.  Measured on MI355X
// (256-session cohorts, W = 32, every launch streaming from HBM): 4-15%
// faster than the two-role split from 1 to 256 workgroups with mod-R
// routes, 5-27% faster at every size with CDF routes; with mod-R routes
// beyond one workgroup per CU it ties or loses (the 100,000-session chain:
// 16.3-16.6 against 14.8-15.4 us).  At W = 16 against the one-lane chain
// (64-session cohorts, T = 8, mod-16 routes): one cohort 6.42 -> 4.82 us,
// 1,000 cohorts in 250 workgroups 8.55 -> 6.5 us.
bool use_piped(uint32_t wmax, bool full, int route_kind, uint32_t grid, uint32_t n_cu) {
    return has_piped(wmax, full) && (grid <= n_cu || route_kind == RK_CDF);
}

template <int WMAX, bool EXACT>
BodyFn body_fn(int body) {
    return body == BODY_BOTH ? rc_body_kernel<WMAX, EXACT, BODY_BOTH>
         : body == BODY_TAKEN ? rc_body_kernel<WMAX, EXACT, BODY_TAKEN>
                              : rc_body_kernel<WMAX, EXACT, BODY_NOT>;
}

BodyFn pick_body(uint32_t wmax, bool exact, int body) {
    switch (wmax) {
        case 4: return exact ? body_fn<4, true>(body) : body_fn<4, false>(body);
        case 8: return exact ? body_fn<8, true>(body) : body_fn<8, false>(body);
        case 16: return exact ? body_fn<16, true>(body) : body_fn<16, false>(body);
        case 32: return exact ? body_fn<32, true>(body) : body_fn<32, false>(body);
        default: return exact ? body_fn<64, true>(body) : body_fn<64, false>(body);
    }
}

// Restores the caller's current device on scope exit.
struct DeviceGuard {
    int prev = -1;
    bool ok = false;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) { prev = -1; return; }
        ok = (prev == dev) || (hipSetDevice(dev) == hipSuccess);
    }
    ~DeviceGuard() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

uint32_t next_pow2_words(uint32_t w) {
    uint32_t p = 4;
    while (p < w) p <<= 1;
    return p;
}

uint32_t ceil_log2(uint32_t x) {
    uint32_t g = 0;
    while ((1u << g) < x) ++g;
    return g;
}

// Validated buffer sets remembered per handle (see validate_buffers).
constexpr int EXTENT_CACHE = 16;
struct BufferKey {
    const void* p[7];
    uint64_t bytes[7];
    bool operator==(const BufferKey& o) const {
        for (int i = 0; i < 7; ++i)
            if (p[i] != o.p[i] || bytes[i] != o.bytes[i]) return false;
        return true;
    }
};

}  // namespace

struct rc_cohort {
    int device = -1;
    uint32_t N = 0, W = 0, R = 0, C = 0, thr = 0;
    RouteArgs ra{};
    uint32_t wmax = 4;
    bool exact = true;
    bool full = true;
    int route_kind = 0;  // RK_POW2 / RK_MOD / RK_CDF
    uint32_t nwave = 4;
    uint32_t img_words = 0, tools_off = 0, cdf_off = 0, guide_off = 0, rows_off = 0, chain_words = 0;
    size_t chain_lds_bytes = 0;
    uint32_t chain_threads = 256;  // threads of a chain workgroup
    std::vector<uint32_t> offsets;  // host copy [C+1]
    Plan plan;
    // All device memory of the handle is one allocation (see rc_cohort_create).
    char* d_block = nullptr;
    uint32_t* d_offsets = nullptr;
    uint32_t* d_raw = nullptr;
    uint32_t* d_cdf = nullptr;
    uint32_t* d_img = nullptr;
    uint32_t* d_wdesc = nullptr;
    uint2* d_lane_i = nullptr;     // plan lanes (see rc_lanes_kernel)
    uint32_t* d_lane_s = nullptr;
    uint32_t table_wgs = 256;      // table image: workgroups that fit the device at once
    uint32_t* d_where = nullptr;  // host round trip: [N] session -> slot | d << 31
    uint32_t* d_ctr = nullptr;
    uint32_t* h_word = nullptr;  // pinned
    uint32_t parity = 0;
    bool ctr_dirty = false;
    uint32_t last_launches = 0, last_d2h = 0;
    // Recorded after the last body kernel of a host-round-trip call; the next
    // such call's stream waits for it before touching d_where / d_ctr.
    hipEvent_t hrt_done = nullptr;
    bool hrt_pending = false;
    uint32_t n_cu = 256;             // compute units of the device
    size_t lds_per_cu = 160u * 1024u;
    BufferKey seen[EXTENT_CACHE];    // buffer sets that passed the device checks
    int n_seen = 0, next_seen = 0;
};

namespace {

void free_handle(rc_cohort* h) {
    if (!h) return;
    if (h->device >= 0) {
        DeviceGuard g(h->device);
        (void)hipFree(h->d_block);
        if (h->h_word) (void)hipHostFree(h->h_word);
        if (h->hrt_done) (void)hipEventDestroy(h->hrt_done);
    }
    delete h;
}

// Per device: the address of rc_noalloc_scratch (resolved once, with the
// device current) and the event that orders the no-allocation
// host-round-trip calls that share it.
constexpr int MAX_DEVICES = 64;
std::mutex g_noalloc_mu;
uint32_t* g_noalloc_ptr[MAX_DEVICES] = {};
hipEvent_t g_noalloc_done[MAX_DEVICES] = {};
bool g_noalloc_pending[MAX_DEVICES] = {};

// Called by rc_cohort_create with `dev` current.
int noalloc_init(int dev) {
    if (dev < 0 || dev >= MAX_DEVICES) return RC_E_DEVICE;
    std::lock_guard<std::mutex> lk(g_noalloc_mu);
    if (g_noalloc_ptr[dev]) return RC_OK;
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(rc_noalloc_scratch)) != hipSuccess || !ptr) {
        (void)hipGetLastError();
        return RC_E_DEVICE;
    }
    hipEvent_t ev = nullptr;
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        return RC_E_DEVICE;
    }
    g_noalloc_done[dev] = ev;
    g_noalloc_ptr[dev] = static_cast<uint32_t*>(ptr);
    return RC_OK;
}

int dev_upload(uint32_t* dst, const uint32_t* src, size_t words) {
    return !words || hipMemcpy(dst, src, words * 4u, hipMemcpyHostToDevice) == hipSuccess ? RC_OK : RC_E_DEVICE;
}

// Is [p, p + bytes) inside one HIP allocation of device `dev`?
bool device_extent_ok(const void* p, size_t bytes, int dev) {
    if (!p) return false;
    hipPointerAttribute_t attr;
    if (hipPointerGetAttributes(&attr, p) != hipSuccess) { (void)hipGetLastError(); return false; }
    if (attr.type != hipMemoryTypeDevice && attr.type != hipMemoryTypeManaged) return false;
    if (attr.device != dev) return false;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p) != hipSuccess) { (void)hipGetLastError(); return false; }
    const uintptr_t b = (uintptr_t)base, q = (uintptr_t)p;
    return q >= b && q - b <= size && bytes <= size - (q - b);
}

// The caller's buffers (and, for the no-decision floor, its decision
// bitmap): present, pairwise disjoint, and each inside one device allocation
// of the handle's device.  The allocation check queries the HIP runtime; a
// buffer set (pointers and extents) that passed it is remembered, and the
// last EXTENT_CACHE such sets are not queried again.
int validate_buffers(rc_cohort* h, const rc_buffers* b, uint32_t T, bool floor = false,
                     const uint32_t* dbits = nullptr) {
    if (!b) return RC_E_INVALID;
    if (b->ld < h->N || b->ld > RC_MAX_SESSIONS) return RC_E_INVALID;
    const uint64_t ld = b->ld;
    struct Ext { const void* p; uint64_t bytes; } ext[7] = {
        {b->state, 4ull * h->W * ld},
        {b->outcome, 4ull * ld},
        {b->eff_sid, 4ull * T * ld},
        {b->eff_tool, 4ull * T * ld},
        {b->eff_payload, 16ull * T * ld},
        {b->n_taken, 4ull * T * h->C},
        {dbits, 4ull * T * ((ld + 31u) / 32u)},
    };
    const int n = floor ? 7 : 6;
    for (int i = 0; i < n; ++i) {
        if (!ext[i].p) return RC_E_INVALID;
        if (ext[i].bytes >= (1ull << 46)) return RC_E_INVALID;
    }
    for (int i = 0; i < n; ++i)
        for (int j = i + 1; j < n; ++j) {
            const uintptr_t a0 = (uintptr_t)ext[i].p, a1 = a0 + ext[i].bytes;
            const uintptr_t b0 = (uintptr_t)ext[j].p, b1 = b0 + ext[j].bytes;
            if (a0 < b1 && b0 < a1) return RC_E_INVALID;
        }
    BufferKey key;
    for (int i = 0; i < 7; ++i) {
        key.p[i] = i < n ? ext[i].p : nullptr;
        key.bytes[i] = i < n ? ext[i].bytes : 0u;
    }
    for (int i = 0; i < h->n_seen; ++i)
        if (h->seen[i] == key) return RC_OK;
    for (int i = 0; i < n; ++i)
        if (ext[i].bytes && !device_extent_ok(ext[i].p, ext[i].bytes, h->device)) return RC_E_INVALID;
    h->seen[h->next_seen] = key;
    h->next_seen = (h->next_seen + 1) % EXTENT_CACHE;
    if (h->n_seen < EXTENT_CACHE) ++h->n_seen;
    return RC_OK;
}

int launch_ok() {
    return hipGetLastError() == hipSuccess ? RC_OK : RC_E_DEVICE;
}

// Table image: persistent workgroups, as many as fit the device at once.
int run_table(rc_cohort* h, const rc_buffers* b, uint32_t step0, uint32_t T, uint32_t cb, uint32_t ce,
              hipStream_t stream, const uint32_t* dbits) {
    TableArgs a;
    a.state = b->state;
    a.outcome = b->outcome;
    a.eff_sid = b->eff_sid;
    a.eff_tool = b->eff_tool;
    a.eff_payload = b->eff_payload;
    a.n_taken = b->n_taken;
    a.img = h->d_img;
    a.lane_s = h->d_lane_s;
    a.lane_i = h->d_lane_i;
    a.ra = h->ra;
    a.ld = b->ld;
    a.n_words = h->W;
    a.n_cohorts = h->C;
    a.thr = h->thr;
    a.step0 = step0;
    a.n_steps = T;
    a.s_lo = h->offsets[cb];
    a.s_n = h->offsets[ce] - a.s_lo;
    uint32_t b_n;
    bins_of_range(h->plan, cb, ce, a.bins_a_lo, a.bins_a_n, a.bins_b_lo, b_n);
    a.n_units = a.bins_a_n + b_n;
    a.img_words = h->img_words;
    a.chain_words = h->chain_words;
    a.cdf_off = h->cdf_off;
    a.guide_off = h->guide_off;
    a.zero_row = table_row_field(h->rows_off, h->R);
    a.dbits = dbits;
    a.dwords = (b->ld + 31u) / 32u;
    const uint32_t grid = a.n_units < h->table_wgs ? a.n_units : h->table_wgs;
    TableFn fn = pick_table((h->W + 15u) / 16u, h->route_kind, dbits != nullptr);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(1024), h->chain_lds_bytes, stream, a);
    if (launch_ok() != RC_OK) return RC_E_DEVICE;
    h->last_launches = 1;
    h->last_d2h = 0;
    return RC_OK;
}

int run_resident(rc_cohort* h, const rc_buffers* b, uint32_t step0, uint32_t T,
                 uint32_t cb, uint32_t ce, hipStream_t stream, const uint32_t* dbits = nullptr) {
    if (!h->full) return run_table(h, b, step0, T, cb, ce, stream, dbits);
    ChainArgs a;
    a.state = b->state;
    a.outcome = b->outcome;
    a.eff_sid = b->eff_sid;
    a.eff_tool = b->eff_tool;
    a.eff_payload = b->eff_payload;
    a.n_taken = b->n_taken;
    a.img = h->d_img;
    a.wdesc = h->d_wdesc;
    a.lane_s = h->d_lane_s;
    a.lane_i = h->d_lane_i;
    a.ra = h->ra;
    a.ld = b->ld;
    a.n_words = h->W;
    a.n_cohorts = h->C;
    a.thr = h->thr;
    a.step0 = step0;
    a.n_steps = T;
    a.s_lo = h->offsets[cb];
    a.s_n = h->offsets[ce] - a.s_lo;
    bins_of_range(h->plan, cb, ce, a.bins_a_lo, a.bins_a_n, a.bins_b_lo, a.bins_b_n);
    a.img_words = h->img_words;
    a.tools_off = h->tools_off;
    a.cdf_off = h->cdf_off;
    a.guide_off = h->guide_off;
    a.rows_off = h->rows_off;
    a.chain_words = h->chain_words;
    a.dbits = dbits;
    a.dwords = (b->ld + 31u) / 32u;
    const uint32_t grid = a.bins_a_n + a.bins_b_n;  // one workgroup per bin
    const bool piped = use_piped(h->wmax, h->full, h->route_kind, grid, h->n_cu);
    ChainFn fn = pick_chain(h->wmax, h->exact, piped, h->route_kind, dbits != nullptr);
    // the pipelined split runs three lanes per session, the two-role split two
    hipLaunchKernelGGL(fn, dim3(grid), dim3(piped ? 3u * 64u * h->nwave : h->chain_threads), h->chain_lds_bytes,
                       stream, a);
    if (launch_ok() != RC_OK) return RC_E_DEVICE;
    h->last_launches = 1;
    h->last_d2h = 0;
    return RC_OK;
}

// Where a host-round-trip call keeps its per-step scratch: the slot of
// every stepped session (session s at where[s - lo]), the two counter words of
// the 4-byte observation, and the event that orders the calls sharing them.
struct HrtScratch {
    uint32_t* where;
    uint32_t* ctr;
    uint32_t* parity;   // which counter word the next step adds to
    hipEvent_t done;    // recorded after a call's last body kernel
    bool* pending;      // `done` has been recorded
    bool clear_first;   // clear both counter words with a kernel first
};

int run_host_roundtrip(rc_cohort* h, const rc_buffers* b, uint32_t step0, uint32_t T,
                       uint32_t cb, uint32_t ce, hipStream_t stream, const HrtScratch& sc) {
    uint32_t launches = 0, copies = 0;
    // the previous call that used this scratch may still be running on
    // another stream: wait for its last body kernel
    if (*sc.pending && hipStreamWaitEvent(stream, sc.done, 0) != hipSuccess) return RC_E_DEVICE;
    if (sc.clear_first) {
        hipLaunchKernelGGL(rc_clear_kernel, dim3(1), dim3(64), 0, stream, sc.ctr, 2u);
        if (launch_ok() != RC_OK) return RC_E_DEVICE;
        ++launches;
        *sc.parity = 0;
    }
    uint32_t a_lo, a_n, b_lo, b_n;
    bins_of_range(h->plan, cb, ce, a_lo, a_n, b_lo, b_n);
    const uint32_t units = a_n + b_n;
    const bool few = decide_few(units, h->thr);
    const uint32_t per = !few ? 1u : units < 4u ? units : 4u, wgs = (units + per - 1u) / per;
    const uint32_t grid = few && wgs > DECIDE_WGS ? DECIDE_WGS : wgs;
    const uint32_t lo = h->offsets[cb], hi = h->offsets[ce];
    const uint32_t n_range = hi - lo;
    const uint32_t body_grid = (n_range + 255u) / 256u;
    for (uint32_t t = 0; t < T; ++t) {
        if (!sc.clear_first) h->ctr_dirty = true;  // the handle's counters; cleared again when the step completes
        DecideArgs d;
        d.state = b->state;
        d.outcome = b->outcome;
        d.n_taken = b->n_taken;
        d.where = sc.where;
        d.ctr = sc.ctr;
        d.lane_s = h->d_lane_s;
        d.lane_i = h->d_lane_i;
        d.thr = h->thr;
        d.step = step0 + t;
        d.t_index = t;
        d.n_cohorts = h->C;
        d.s_n = n_range;
        d.bins_a_lo = a_lo;
        d.bins_a_n = a_n;
        d.bins_b_lo = b_lo;
        d.n_units = units;
        d.parity = *sc.parity;
        d.where_lo = lo;
        hipLaunchKernelGGL(rc_decide_kernel, dim3(grid), dim3(per * 256u), 0, stream, d);
        if (launch_ok() != RC_OK) return RC_E_DEVICE;
        ++launches;
        // the observation: 4 bytes to pinned host memory, then wait
        if (hipMemcpyAsync(h->h_word, sc.ctr + *sc.parity, sizeof(uint32_t),
                           hipMemcpyDeviceToHost, stream) != hipSuccess) return RC_E_DEVICE;
        ++copies;
        if (hipStreamSynchronize(stream) != hipSuccess) return RC_E_DEVICE;
        const uint32_t n_taken_total = *h->h_word;
        if (n_taken_total > n_range) return RC_E_DEVICE;
        // the host branch: launch the selected route body, or both in one
        BodyArgs ba;
        ba.state = b->state;
        ba.outcome = b->outcome;
        ba.eff_sid = b->eff_sid;
        ba.eff_tool = b->eff_tool;
        ba.eff_payload = b->eff_payload;
        ba.where = sc.where;
        ba.raw = h->d_raw;
        ba.cdf = h->d_img + h->cdf_off;
        ba.guide = h->d_img + h->guide_off;
        ba.ra = h->ra;
        ba.ld = b->ld;
        ba.n_words = h->W;
        ba.lo = lo;
        ba.hi = hi;
        ba.t_index = t;
        const int body = n_taken_total == 0u ? BODY_NOT : n_taken_total == n_range ? BODY_TAKEN : BODY_BOTH;
        hipLaunchKernelGGL(pick_body(h->wmax, h->exact, body), dim3(body_grid), dim3(256), 0, stream, ba);
        if (launch_ok() != RC_OK) return RC_E_DEVICE;
        ++launches;
        *sc.parity ^= 1u;
        if (!sc.clear_first) h->ctr_dirty = false;
    }
    if (hipEventRecord(sc.done, stream) != hipSuccess) return RC_E_DEVICE;
    *sc.pending = true;
    h->last_launches = launches;
    h->last_d2h = copies;
    return RC_OK;
}

// The handle's own scratch (d_where, d_ctr), after restoring cleared counters
// if a previous call stopped inside a step.
int run_host_roundtrip_handle(rc_cohort* h, const rc_buffers* b, uint32_t step0, uint32_t T,
                              uint32_t cb, uint32_t ce, hipStream_t stream) {
    if (h->ctr_dirty) {
        if (h->hrt_pending && hipStreamWaitEvent(stream, h->hrt_done, 0) != hipSuccess) return RC_E_DEVICE;
        if (hipMemsetAsync(h->d_ctr, 0, 2 * sizeof(uint32_t), stream) != hipSuccess) return RC_E_DEVICE;
        h->parity = 0;
        h->ctr_dirty = false;
    }
    HrtScratch sc{h->d_where + h->offsets[cb], h->d_ctr, &h->parity, h->hrt_done, &h->hrt_pending, false};
    return run_host_roundtrip(h, b, step0, T, cb, ce, stream, sc);
}

}  // namespace

extern "C" {

int rc_cohort_create(const rc_cohort_desc* desc, int hip_device, rc_cohort** out) {
    if (!out) return RC_E_INVALID;
    const int v = validate_desc(desc);
    if (v != RC_OK) return v;

    int n_dev = 0;
    if (hipGetDeviceCount(&n_dev) != hipSuccess || n_dev <= 0) { (void)hipGetLastError(); return RC_E_DEVICE; }
    if (hip_device < 0 || hip_device >= n_dev) return RC_E_DEVICE;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, hip_device) != hipSuccess) return RC_E_DEVICE;
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) return RC_E_DEVICE;
    if (prop.multiProcessorCount < 1 || prop.maxSharedMemoryPerMultiProcessor < 64u * 1024u) return RC_E_DEVICE;

    rc_cohort* h = new (std::nothrow) rc_cohort();
    if (!h) return RC_E_NOMEM;
    DeviceGuard guard(hip_device);
    if (!guard.ok) { delete h; return RC_E_DEVICE; }
    h->device = hip_device;
    h->n_cu = (uint32_t)prop.multiProcessorCount;
    h->lds_per_cu = prop.maxSharedMemoryPerMultiProcessor;
    // the full mask image up to 45% of a CU's LDS (72 KB of 160 KB); two
    // workgroups per CU below half of it
    const size_t full_image_limit = h->lds_per_cu * 9u / 20u;
    const size_t lds_two_per_cu = h->lds_per_cu / 2u;
    h->N = desc->n_sessions;
    h->W = desc->n_words;
    h->R = desc->n_routes;
    h->C = desc->n_cohorts;
    h->thr = desc->decide_thr;
    h->wmax = next_pow2_words(h->W);
    h->exact = (h->wmax == h->W);
    const uint32_t R = h->R;
    // with a single route both route maps give route 0
    h->ra.mode = (desc->route_mode == RC_ROUTE_CDF && R > 1u) ? RC_ROUTE_CDF : RC_ROUTE_MOD;
    h->ra.n_routes = R;
    h->ra.is_pow2 = (R & (R - 1u)) == 0u;
    h->ra.pow2_mask = h->ra.is_pow2 ? R - 1u : 0u;
    h->ra.cdf_n = (h->ra.mode == RC_ROUTE_CDF) ? R - 1u : 0u;
    h->route_kind = h->ra.mode == RC_ROUTE_CDF ? RK_CDF : (h->ra.is_pow2 ? RK_POW2 : RK_MOD);
    h->ra.mod_recip = R > 1u ? (uint32_t)((1ull << 32) / R) : 0u;

    // table image layout (see the file comment)
    const size_t full_bytes = (size_t)(R + 1u) * (h->wmax + 4u) * 4u;
    h->full = h->wmax <= 16u || full_bytes <= full_image_limit;
    // Full image: [word-0 masks | CDF thresholds | guide] (the chain
    // section, everything the word-0 chain reads), then the mask rows, then
    // the tool pairs.  Table image: [route pairs | thresholds | guide], then
    // the raw rows at a multiple of 16 words.
    const uint32_t nb = (h->W + 15u) / 16u;
    const uint32_t row_words = h->full ? h->wmax : 16u;
    const uint32_t tab_words = (R + 1u) * (h->full ? row_words + 4u : row_words);
    auto pad4 = [](uint32_t x) { return (x + 3u) & ~3u; };
    auto pad16 = [](uint32_t x) { return (x + 15u) & ~15u; };
    const uint32_t m0_words = h->full ? pad4(R + 1u) : pad4(2u * R);
    h->cdf_off = m0_words;
    h->guide_off = h->cdf_off + (h->ra.cdf_n ? pad4(h->ra.cdf_n + CDF_PAD) : 0u);
    const uint32_t after_guide = tab_words + (h->full ? pad4(R) : 12u);  // rows and tools (or the rows' alignment)
    // The chain kernel's LDS after the image (full image): the count exchange
    // ([16][nwave + 4] words), then (WMAX >= 16: the two-role or the
    // pipelined split) the control handed to the replaying lanes, 16 steps of
    // a 4-byte addend and a 4-byte control word per lane, then the effect
    // stage of sub-wavefront bins, 4 + 16 bytes per lane.
    const bool ctl_area = h->wmax >= 16u;
    const uint32_t na = h->nwave * 64u;
    const size_t lds_after_image = h->full ? 16u * (h->nwave + 4u) * 4u + (ctl_area ? 16u * na * 8u : 0u) + na * 20u
                                           : table_lds_after(nb);
    uint32_t guide_bits = 0, guide_n = 0;
    if (h->ra.mode == RC_ROUTE_CDF) {
        // Eight buckets per route, at most 2^12: with skewed routes the
        // thresholds of the light routes crowd into few buckets, and every
        // threshold in a bucket is a dependent LDS step of the chain's search
        // (Zipf(1.1) over 64 routes: at most 1 per bucket, 2 with four
        // buckets per route).  Fewer buckets when that keeps two workgroups
        // on a CU that the smallest guide would allow.
        const uint32_t gmin = ceil_log2(R) < 1u ? 1u : ceil_log2(R);
        guide_bits = gmin + 3u < 12u ? gmin + 3u : (gmin > 12u ? gmin : 12u);
        auto lds_at = [&](uint32_t gb) {
            return ((size_t)h->guide_off + pad4((1u << gb) + 1u) + after_guide) * 4u + lds_after_image;
        };
        const size_t lds_goal = lds_at(gmin) <= lds_two_per_cu ? lds_two_per_cu : h->lds_per_cu;
        while (guide_bits > gmin && lds_at(guide_bits) > lds_goal) --guide_bits;
        guide_n = (1u << guide_bits) + 1u;
        h->ra.guide_shift = 32u - guide_bits;
    }
    const uint32_t guide_end = h->guide_off + pad4(guide_n);
    h->chain_words = guide_end;
    h->rows_off = h->full ? guide_end : pad16(guide_end);
    h->tools_off = h->rows_off + tab_words;
    h->img_words = h->full ? h->tools_off + pad4(R) : h->rows_off + tab_words;
    const size_t lds_image = (size_t)h->img_words * 4u;
    // chain_threads is the two-role (W >= 32) or one-lane workgroup; the
    // pipelined split launches three lanes per session.
    const bool split = h->full && h->wmax >= 32u;
    h->chain_threads = (split ? 2u : 1u) * na;
    h->chain_lds_bytes = lds_image + lds_after_image;

    try {
        h->offsets.assign(desc->cohort_offsets, desc->cohort_offsets + h->C + 1u);
        build_plan(h->offsets.data(), h->C, h->nwave, h->plan);
    } catch (const std::bad_alloc&) {
        free_handle(h);
        return RC_E_NOMEM;
    }

    // One device allocation for everything the handle holds, in parts that
    // start at multiples of 256 bytes.  An allocation and its release cost the
    // host little where they are small, but about 40 us together from a few
    // MiB up, and the release after a create that also cleared words with two
    // memsets waited 20 to 40 us: create and destroy of 1,000 sessions took
    // 92 + 75 us with an allocation for each array and two memsets, 77 + 28 us
    // so; of a million sessions 276 + 116 us, 260 + 41 us.
    size_t block_bytes = 0;
    auto part = [&](size_t bytes) {
        const size_t at = block_bytes;
        block_bytes += (bytes + 255u) & ~(size_t)255u;
        return at;
    };
    const size_t lanes = (size_t)h->plan.n_bins * na;
    const size_t at_lane_i = part(lanes * sizeof(uint2));
    const size_t at_lane_s = part(lanes * 4u);
    const size_t at_where = part((size_t)h->N * 4u);
    const size_t at_wdesc = part(h->plan.wdesc.size() * 4u);
    const size_t at_offsets = part(h->offsets.size() * 4u);
    const size_t at_raw = part((size_t)R * 16u * 4u);
    const size_t at_cdf = part((size_t)h->ra.cdf_n * 4u);
    const size_t at_img = part((size_t)h->img_words * 4u);
    const size_t at_words = part(3u * 4u);  // two counters, then the largest guide bucket span
    int rc = hipMalloc((void**)&h->d_block, block_bytes) == hipSuccess ? RC_OK : RC_E_NOMEM;
    if (rc == RC_OK) {
        auto words_at = [&](size_t at) { return reinterpret_cast<uint32_t*>(h->d_block + at); };
        h->d_lane_i = reinterpret_cast<uint2*>(h->d_block + at_lane_i);
        h->d_lane_s = words_at(at_lane_s);
        h->d_where = words_at(at_where);
        h->d_wdesc = words_at(at_wdesc);
        h->d_offsets = words_at(at_offsets);
        h->d_raw = words_at(at_raw);
        h->d_cdf = words_at(at_cdf);
        h->d_img = words_at(at_img);
        h->d_ctr = words_at(at_words);
    }
    if (rc == RC_OK) rc = dev_upload(h->d_offsets, h->offsets.data(), h->offsets.size());
    if (rc == RC_OK) rc = dev_upload(h->d_raw, desc->table, (size_t)R * 16u);
    if (rc == RC_OK) rc = dev_upload(h->d_cdf, desc->route_cdf, h->ra.cdf_n);
    if (rc == RC_OK) rc = dev_upload(h->d_wdesc, h->plan.wdesc.data(), h->plan.wdesc.size());
    if (rc == RC_OK && hipHostMalloc((void**)&h->h_word, sizeof(uint32_t), hipHostMallocDefault) != hipSuccess) rc = RC_E_NOMEM;
    if (rc == RC_OK && hipEventCreateWithFlags(&h->hrt_done, hipEventDisableTiming) != hipSuccess) rc = RC_E_DEVICE;
    if (rc == RC_OK) rc = noalloc_init(hip_device);
    if (rc == RC_OK) {
        hipLaunchKernelGGL(rc_lanes_kernel, dim3(h->plan.n_bins), dim3(na), 0, 0, h->d_wdesc, h->d_offsets,
                           h->d_lane_s, h->d_lane_i, h->d_ctr, 3u);
        rc = launch_ok();
    }
    if (rc == RC_OK) {
        ImageArgs ia;
        ia.raw = h->d_raw;
        ia.cdf = h->d_cdf;
        ia.img = h->d_img;
        ia.max_span = h->d_ctr + 2;
        ia.n_routes = R;
        ia.row_words = row_words;
        ia.full = h->full ? 1u : 0u;
        ia.tab_words = tab_words;
        ia.tools_off = h->tools_off;
        ia.cdf_off = h->cdf_off;
        ia.cdf_n = h->ra.cdf_n;
        ia.guide_off = h->guide_off;
        ia.guide_n = guide_n;
        ia.guide_shift = h->ra.guide_shift;
        ia.total_words = h->img_words;
        ia.m0_words = m0_words;
        ia.rows_off = h->rows_off;
        hipLaunchKernelGGL(rc_prep_kernel, dim3((h->img_words + 255u) / 256u), dim3(256), 0, 0, ia);
        uint32_t span = 0;
        // the copy waits for both kernels: callers' streams need not
        if (launch_ok() != RC_OK || hipMemcpy(&span, h->d_ctr + 2, 4, hipMemcpyDeviceToHost) != hipSuccess)
            rc = RC_E_DEVICE;
        h->ra.guide_top = 0;
        while (span && (h->ra.guide_top << 1) <= span) h->ra.guide_top = h->ra.guide_top ? h->ra.guide_top << 1 : 1u;
    }
    for (int v = 0; v < 4 && rc == RC_OK; ++v) {
        const bool fl = (v & 1) != 0, piped = (v & 2) != 0;
        if (piped && !has_piped(h->wmax, h->full)) continue;
        const void* fn = h->full ? (const void*)pick_chain(h->wmax, h->exact, piped, h->route_kind, fl)
                                 : (const void*)pick_table(nb, h->route_kind, fl);
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)h->chain_lds_bytes) != hipSuccess)
            rc = RC_E_DEVICE;
        int per_cu = 0;
        if (rc == RC_OK && !h->full && !fl) {
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 1024, h->chain_lds_bytes) != hipSuccess ||
                per_cu < 1) rc = RC_E_DEVICE;
            h->table_wgs = h->n_cu * (uint32_t)per_cu;
        }
    }
    if (rc != RC_OK) {
        (void)hipGetLastError();
        free_handle(h);
        return rc;
    }
    *out = h;
    return RC_OK;
}

int rc_cohort_run_chain(rc_cohort* h, const rc_buffers* b, uint32_t step0, uint32_t n_steps,
                        int mode, uint32_t cohort_begin, uint32_t cohort_end, void* hip_stream) {
    if (!h || !b) return RC_E_INVALID;
    if (mode != RC_MODE_RESIDENT && mode != RC_MODE_HOST_ROUNDTRIP) return RC_E_INVALID;
    if (cohort_begin > cohort_end || cohort_end > h->C) return RC_E_INVALID;
    DeviceGuard guard(h->device);
    if (!guard.ok) return RC_E_DEVICE;
    const int v = validate_buffers(h, b, n_steps);
    if (v != RC_OK) return v;
    h->last_launches = 0;
    h->last_d2h = 0;
    if (n_steps == 0u || cohort_begin == cohort_end) return RC_OK;
    hipStream_t stream = (hipStream_t)hip_stream;
    if (mode == RC_MODE_RESIDENT) return run_resident(h, b, step0, n_steps, cohort_begin, cohort_end, stream);
    return run_host_roundtrip_handle(h, b, step0, n_steps, cohort_begin, cohort_end, stream);
}

int rc_cohort_run_chain_noalloc(rc_cohort* h, const rc_buffers* b, uint32_t step0, uint32_t n_steps,
                                int mode, uint32_t cohort_begin, uint32_t cohort_end, void* hip_stream) {
    if (!h || !b) return RC_E_INVALID;
    if (mode != RC_MODE_RESIDENT && mode != RC_MODE_HOST_ROUNDTRIP) return RC_E_INVALID;
    if (cohort_begin > cohort_end || cohort_end > h->C) return RC_E_INVALID;
    if (h->offsets[cohort_end] - h->offsets[cohort_begin] > RC_NOALLOC_MAX_SESSIONS) return RC_E_INVALID;
    DeviceGuard guard(h->device);
    if (!guard.ok) return RC_E_DEVICE;
    const int v = validate_buffers(h, b, n_steps);
    if (v != RC_OK) return v;
    h->last_launches = 0;
    h->last_d2h = 0;
    if (n_steps == 0u || cohort_begin == cohort_end) return RC_OK;
    hipStream_t stream = (hipStream_t)hip_stream;
    // the resident chain uses no scratch
    if (mode == RC_MODE_RESIDENT) return run_resident(h, b, step0, n_steps, cohort_begin, cohort_end, stream);
    uint32_t* base = g_noalloc_ptr[h->device];  // resolved by rc_cohort_create
    if (!base) return RC_E_DEVICE;
    uint32_t parity = 0;
    HrtScratch sc{base + NOALLOC_WHERE_OFF, base, &parity, g_noalloc_done[h->device],
                  &g_noalloc_pending[h->device], true};
    return run_host_roundtrip(h, b, step0, n_steps, cohort_begin, cohort_end, stream, sc);
}

int rc_cohort_run_floor(rc_cohort* h, const rc_buffers* b, const uint32_t* decisions, uint32_t n_steps,
                        uint32_t cohort_begin, uint32_t cohort_end, void* hip_stream) {
    if (!h || !b || !decisions) return RC_E_INVALID;
    if (cohort_begin > cohort_end || cohort_end > h->C) return RC_E_INVALID;
    DeviceGuard guard(h->device);
    if (!guard.ok) return RC_E_DEVICE;
    const int v = validate_buffers(h, b, n_steps, true, decisions);
    if (v != RC_OK) return v;
    h->last_launches = 0;
    h->last_d2h = 0;
    if (n_steps == 0u || cohort_begin == cohort_end) return RC_OK;
    return run_resident(h, b, 0u, n_steps, cohort_begin, cohort_end, (hipStream_t)hip_stream, decisions);
}

int rc_cohort_step(rc_cohort* h, const rc_buffers* b, uint32_t step, uint32_t cohort_begin,
                   uint32_t cohort_end, void* hip_stream) {
    return rc_cohort_run_chain(h, b, step, 1u, RC_MODE_RESIDENT, cohort_begin, cohort_end, hip_stream);
}

int rc_cohort_destroy(rc_cohort* h) {
    free_handle(h);
    return RC_OK;
}

int rc_cohort_last_counts(const rc_cohort* h, uint32_t* launches, uint32_t* d2h_copies) {
    if (!h) return RC_E_INVALID;
    if (launches) *launches = h->last_launches;
    if (d2h_copies) *d2h_copies = h->last_d2h;
    return RC_OK;
}

int rc_cohort_plan_info(const rc_cohort* h, uint32_t* n_workgroups, uint32_t* lanes_per_workgroup,
                        uint32_t* idle_lanes) {
    if (!h) return RC_E_INVALID;
    if (n_workgroups) *n_workgroups = h->plan.n_bins;
    if (lanes_per_workgroup) *lanes_per_workgroup = h->nwave * 64u;
    if (idle_lanes) *idle_lanes = h->plan.idle_lanes;
    return RC_OK;
}

}  // extern "C"

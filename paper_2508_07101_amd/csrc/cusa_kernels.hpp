// Device code of libcusa: gfx950 kernels for the CUSA decode hot path.
//
//   topk_kernel         per-head ranked top-k (Sec. 3.2): a threshold from a sample, one compare per
//                       score, a counting sort over value bins of what passes (rank_entries); radix select
//                       and a bitonic sort held in registers for rows where that does not work out
//   slice_filter_kernel the same threshold on slices of few long rows
//   union_kernel        cross-head union, first-occurrence global rank, cut at
//                       K-W, recency window (Sec. 3.2, 3.3) -> ascending rho
//   score_kernel        P = q.K^T (Alg. 1, selection layer): one lane per key row, K staged
//                       through LDS, products accumulated by k = 1 MFMA in column order
//   topk_values_kernel  a selection layer's top-k and, on the rest of the chip, its output
//                       softmax(P) V from those scores
//   attn_kernel         split-K flash-decode over all tokens or over rho
//                       (Eq. 1 / SparseAttention of Alg. 1), GQA group in registers; its scoring
//                       forms also write the candidates' scores, or keep those above a threshold
//   sample_threshold_kernel   per-head thresholds from a sample of the scores (filtered selection)
//   attn_reduce_kernel  merges the split-K partials and writes bf16
//   per_head_rho_kernel, rank_aggregate_kernel, recall_kernel   the head-to-head variant, the other
//                       two readings of the global ranking, the recall of Eq. 3
//   probe_*_kernel      traffic probes (benchmark support)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_plan.hpp"

namespace cusa {

constexpr int D = 128;        // head_dim
constexpr int PAGE = 16;      // tokens per page of a paged cache

struct KvView {
    const uint16_t* k;
    const uint16_t* v;
    int64_t sb, sh, st;       // contiguous: element strides (batch, kv head, token)
    const int32_t* bt;        // paged: block table [B][max_pages]
    int32_t max_pages;
    int32_t G;                // kv heads
    const int32_t* seq_lens;  // [B]
};

template <bool PAGED>
__device__ __forceinline__ int64_t row_offset(const KvView& kv, int b, int kvh, int pos) {
    if (PAGED) {
        int64_t page = kv.bt[(int64_t)b * kv.max_pages + (pos >> 4)];
        return ((page * kv.G + kvh) * PAGE + (pos & (PAGE - 1))) * D;
    }
    return (int64_t)b * kv.sb + (int64_t)kvh * kv.sh + (int64_t)pos * kv.st;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// 16 bytes of a K or V row.  Every row is read once per pass, so the load carries the streaming
// (non-temporal) hint: the caches need not keep what will not be asked for again.  On this machine that
// is worth 7-11 % on every attention kernel (c3 full attention 90 -> 83 us, c5 sparse 99 -> 88 us): a
// pass no longer turns over the whole L2 with lines nobody returns to.
__device__ __forceinline__ u32x4 stream_load(const uint16_t* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}

// With per-head token lists the heads of a group ask for many of the same rows from different
// workgroups: those loads stay ordinary, so that the second asker finds the row in L2.
template <bool SHARED_ROWS>
__device__ __forceinline__ u32x4 row_load(const uint16_t* p) {
    return SHARED_ROWS ? *reinterpret_cast<const u32x4*>(p) : stream_load(p);
}

// A value at a wave-uniform address that no kernel of the launch writes: a scalar load.
__device__ __forceinline__ int32_t uniform_load(const int32_t* p) {
    return *(const __attribute__((address_space(4))) int32_t*)(uintptr_t)p;
}

// Where a running maximum of scores starts: no score of a tile needs to be finite.  (From -infinity, a first tile whose scores are all
// -infinity makes NaN of its weights; from here they are 2^-infinity = 0.)
constexpr float LOWEST = -3.402823466e38f;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ void unpack8(const uint4& w, float* f) {
    f[0] = bf16_lo(w.x); f[1] = bf16_hi(w.x);
    f[2] = bf16_lo(w.y); f[3] = bf16_hi(w.y);
    f[4] = bf16_lo(w.z); f[5] = bf16_hi(w.z);
    f[6] = bf16_lo(w.w); f[7] = bf16_hi(w.w);
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;   // NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------- scoring
//
// The selection scores P = q.K^T are made by score_kernel and, in the same pass as a selection layer's output or where only candidates above a
// threshold are kept, by attn_kernel's scoring forms.  Their bit-exactness rests on the product
// chain: V_MFMA_F32_4X4X1_16B_F32 takes, per lane, one binary32 element of q (head = lane % 4) and one
// of K (the lane's row) and adds the 4 heads x 64 rows of single products to the accumulators.  With
// k = 1 there is exactly one product (exact: bf16 x bf16 has a 16-bit significand) and one rounded
// addition per instruction, so walking the 128 columns in order is the left-to-right binary32 sum --
// no reordering inside the instruction can occur.  (Checked bit for bit against a scalar fmaf chain
// on the device.)

constexpr int SCORE_ROWS = 64;                        // tokens of a sample tile

// ---------------------------------------------------------------- block helpers

constexpr int SEL_THREADS = 1024;
constexpr int SEL_WAVES = SEL_THREADS / 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }

// number of set bits of a 64-bit ballot below this lane
__device__ __forceinline__ int mbcnt(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// Inclusive prefix sum over a wave by DPP moves: inside the 16-lane rows, then across them.
__device__ __forceinline__ int wave_scan_incl(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
    return v;
}

// Workgroup barrier for data exchanged through LDS only: waits for this wave's LDS operations, not for
// its outstanding global loads (which a full __syncthreads() would drain first).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// LDS written by some lanes of a wave and read by others of the same wave: a wave's LDS
// accesses are performed in program order, so only the compiler has to be kept from
// reordering them.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exclusive prefix sum of one int per thread over a block of WAVES waves.
// scratch: WAVES ints of LDS.  Returns the exclusive prefix; *total gets the sum.
// Every wave adds up the other waves' sums for itself: one wave's lane doing it for all costs as much
// as the rest of the scan.
template <int WAVES = SEL_WAVES>
__device__ __forceinline__ int block_scan_excl(int v, int* scratch, int* total) {
    const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
    const int inc = wave_scan_incl(v);
    lds_barrier();                                 // scratch may still be read from a previous call
    if (lane == 63) scratch[w] = inc;
    lds_barrier();
    int before = 0, sum = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
        const int c = scratch[i];
        before += i < w ? c : 0;
        sum += c;
    }
    *total = sum;
    return before + inc - v;
}

// Order-preserving map of a binary32 score to uint32 (larger score -> larger key);
// -0 is mapped like +0 so that the two compare equal.
__device__ __forceinline__ uint32_t score_key(float s) {
    uint32_t u = __float_as_uint(s);
    if (u == 0x80000000u) u = 0;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// State of the selection's filtered fast path (sample_threshold_kernel has the account).
struct FilterState {              // device memory of the fast path, all per (sequence, head) = row
    uint32_t* thr;                // threshold key; 0xffffffff: keep nothing (flagged, or nothing to select)
    int32_t* cand_cnt;            // candidates kept so far
    int32_t* fail;                // 1: this head takes the second chance
    int32_t* n_failed;            // number of flagged heads
    union {
        uint64_t* cand;           // [row][cap] composites (score key << 32 | ~position), in any order
        float* scores;            // attn_kernel's scoring variant without the filter: P, rows of cap scores.  (Arguments of their own, which
    };                            // every form of the kernel would load: 0.2 us per launch, 401 -> 408 for a step of 36 layers.)
    int32_t cap;
    int32_t n_sink;
};

// Flags are set wherever a head's guess turns out bad; the heads are counted in one place, the top-k over
// the kept candidates, which looks at every head once.
__device__ __forceinline__ void flag_failed(const FilterState& f, int64_t row) { f.fail[row] = 1; }

// Inverse of score_key.
__device__ __forceinline__ float key_score(uint32_t key) {
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// ---------------------------------------------------------------- per-head top-k
//
// One 1024-thread workgroup per (sequence, head).  The candidates are ordered by
// the 64-bit composite (score_key << 32 | ~position): larger composite = better
// score, or equal score and lower position -- a strict total order, so "the k best"
// is a unique set and a unique ranking.
//
// Fast path: a threshold from a sample of the row (sample_row), one look at every score against it, the few
// that pass compacted into one LDS list, and these ranked by a counting sort over value bins
// (rank_entries) -- or, where many of them are equal, sorted.  Ranks are written rank-major: rho_head[b][j][h].
// General path, for rows where that does not work out (scores that are not finite, more passing than the list holds: massive
// ties, thresholds that were no good) and for raw keys:
//   1. radix select (11/11/10-bit digits, LDS histograms) finds the score key T
//      of the k-th best candidate and how many candidates tie with it;
//   2. if more candidates equal T than are still needed, a second radix select
//      over ~position finds the position bound among the ties;
//   3. the k survivors are compacted into LDS and ranked, or bitonic-sorted (descending).
// With ITEMS > 0 a thread keeps ITEMS scores in registers, loaded once with independent 16-byte loads;
// ITEMS <= 0 (streamed) reads the row again in every pass, in batches (any length).
//
// What bounds it: one CU per row, its sixteen waves' instructions (each costs the CU sixteen cycles), the barriers
// between them and, first, the row's way from memory (3 us of the 14 at 32 K candidates).  Measured before (selection
// with digit histograms, then ranking) -> after, us, rows still in the last-level cache (in a step they come from memory: 13.6,
// 15.5 and 33 us for the second, third and fourth size): 32 rows of 3840, k 1024: 7.9 -> 7.7; 32 rows of 32256, k 1536:
// 16.9 -> 11.9; 256 rows of 15360, k 3072: 16.7 -> 13.5; 64 rows of 130048, k 3072, in slices: 36.5 -> 24.1; 576 rows of
// 11552, k 2304: 56.8 -> 25.3; 1408 rows of 22798, k 3072: 145 -> 62.1.  Scores that are correlated over 64 positions each
// take the same times within 1 per cent.

struct SelectState {
    uint32_t prefix;     // digits fixed so far
    int need;            // how many of the candidates matching prefix are wanted
    int count_eq;        // candidates whose digit equals the chosen one (last pass)
};

// One radix-select pass over `hist` (NB bins, already filled): choose the digit
// in which the `need`-th largest lies.  All threads call; results via LDS `st`.
template <int NB>
__device__ __forceinline__ void pick_digit(int* hist, int* scratch, SelectState* st, int shift) {
    // thread i owns bins [i*PER, i*PER+PER) counted from the top (descending digits)
    constexpr int PER = (NB + SEL_THREADS - 1) / SEL_THREADS;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                        // addresses are made here, not kept from far above
    int local[PER];
    int sum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        int bin = NB - 1 - (tid * PER + j);
        local[j] = bin >= 0 ? hist[bin] : 0;
        sum += local[j];
    }
    int total;
    int above = block_scan_excl(sum, scratch, &total);   // candidates with larger digits
    const int need = st->need;
    __syncthreads();                                     // everyone has read st->need
    if (above < need && need <= above + sum) {
        int run = above;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (run < need && need <= run + local[j]) {
                int bin = NB - 1 - (tid * PER + j);
                st->prefix |= (uint32_t)bin << shift;
                st->need = need - run;
                st->count_eq = local[j];
            }
            run += local[j];
        }
    }
    __syncthreads();
}

// Radix select of the `need`-th largest 32-bit key among this workgroup's candidates.
// scan(f) must call f(key, t) for every candidate slot of the calling thread, the same
// number of times in every lane of a wave; slots past the candidate range carry key 0, which
// no real score maps to and which therefore never reaches the top k.  key_map(key, t, &out)
// narrows the candidates and chooses the key that is selected on.
// Leaves the key in st->prefix, the number still wanted among equal keys in st->need and
// their count in st->count_eq.
// Keys whose top digit is below min_digit0 are known not to matter and are not counted.
// first_pass > 0 resumes a selection whose leading digits *st already holds.
template <typename Scan, typename KeyMap>
__device__ __forceinline__ void radix_select(int first_pass, int need, uint32_t min_digit0, Scan scan, KeyMap key_map,
                                             int* hist, int* scratch, SelectState* st) {
    if (first_pass == 0 && threadIdx.x == 0) {
        st->prefix = 0;
        st->need = need;
        st->count_eq = 0;
    }
    const int shifts[3] = {21, 10, 0};
    const int bits[3] = {11, 11, 10};
    uint32_t mask = 0;
    for (int pass = 0; pass < first_pass; ++pass) mask |= ((1u << bits[pass]) - 1u) << shifts[pass];
    for (int pass = first_pass; pass < 3; ++pass) {
        for (int i = threadIdx.x; i < 2048; i += SEL_THREADS) hist[i] = 0;
        __syncthreads();
        const uint32_t prefix = st->prefix;
        const int shift = shifts[pass];
        const uint32_t dmask = (1u << bits[pass]) - 1u;
        const uint32_t floor_d = pass == 0 ? min_digit0 : 0u;
        scan([&](uint32_t skey, int t) {
            uint32_t key;
            if (key_map(skey, t, &key) && (key & mask) == prefix && ((key >> shift) & dmask) >= floor_d)
                atomicAdd(&hist[(key >> shift) & dmask], 1);
        });
        __syncthreads();
        if (pass < 2) pick_digit<2048>(hist, scratch, st, shift);
        else pick_digit<1024>(hist, scratch, st, shift);
        mask |= dmask << shift;
    }
}

// Adds this thread's count to a workgroup counter with one LDS atomic per wave; returns the first of
// the thread's slots.  The counter must be zero and visible before, and is complete after the next
// workgroup barrier.
__device__ __forceinline__ int wave_reserve(int mine, int* counter) {
    const int inc = wave_scan_incl(mine);
    int wave_base = 0;
    if (lane_id() == 63) wave_base = atomicAdd(counter, inc);
    return __builtin_amdgcn_readlane(wave_base, 63) + inc - mine;
}

// Entries of the LDS candidate list of topk_kernel<ITEMS, MTOP> (0: no list; short rows are
// cheap to walk again).
__host__ __device__ constexpr int topk_list_cap(int items, int mtop) {
    return (items > 0 && items < 8) ? 0 : mtop <= 2 ? 6144 : mtop <= 4 ? 5120 : 10240;
}
// Value of lane (l ^ STRIDE) for STRIDE < 64 without the LDS crossbar: DPP moves inside a 16-lane
// row, row/half swaps beyond.
template <int CTRL, int BANK_MASK = 0xF>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, 0xF, BANK_MASK, false);
}
template <int STRIDE>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    // every lane has a source lane, so a plain DPP move into a fresh register does it (one
    // instruction, no copy of the destination's previous value)
    if constexpr (STRIDE == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);        // quad_perm [1,0,3,2]
    else if constexpr (STRIDE == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
    else if constexpr (STRIDE == 4) {
        const uint32_t t = dpp_u32<0x104, 0x5>(v, v);                 // row_shl:4 into lanes 0-3, 8-11 of a row
        return dpp_u32<0x114, 0xA>(t, v);                             // row_shr:4 into lanes 4-7, 12-15
    } else if constexpr (STRIDE == 8) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);   // row_ror:8
    else if constexpr (STRIDE == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);   // s[0]: rows 0,0,2,2; s[1]: rows 1,1,3,3
        return (threadIdx.x & 16) ? s[0] : s[1];
    } else {
        static_assert(STRIDE == 32, "lane_xor: stride must be a power of two below 64");
        const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);   // s[0]: lower half twice; s[1]: upper half twice
        return (threadIdx.x & 32) ? s[0] : s[1];
    }
}
// One step of the bitonic network over MTOP * 1024 composites, MTOP per thread, and all steps after it (see topk_kernel).
template <int MTOP, int SIZE, int STRIDE>
__device__ __forceinline__ void bitonic_sort(uint64_t (&v)[MTOP], uint64_t* sort_buf, int base) {
    if constexpr (STRIDE >= 64 * MTOP) {               // partner in another wave
        __syncthreads();
#pragma unroll
        for (int j = 0; j < MTOP; ++j) sort_buf[base + j * 64] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < MTOP; ++j) {
            const int i = base + j * 64;
            const uint64_t o = sort_buf[i ^ STRIDE];
            const bool keep_max = ((i & STRIDE) == 0) == ((i & SIZE) == 0);
            v[j] = ((v[j] > o) == keep_max) ? v[j] : o;
        }
    } else if constexpr (STRIDE >= 64) {               // partner in this thread's registers
        constexpr int JS = STRIDE >> 6;
#pragma unroll
        for (int j = 0; j < MTOP; ++j) {
            if ((j & JS) == 0 && (j | JS) < MTOP) {
                const bool desc = ((base + j * 64) & SIZE) == 0;
                const uint64_t a = v[j], c = v[j | JS];
                const bool sw = (a < c) == desc;
                v[j] = sw ? c : a;
                v[j | JS] = sw ? a : c;
            }
        }
    } else {                                           // partner in another lane of this wave
#pragma unroll
        for (int j = 0; j < MTOP; ++j) {
            const int i = base + j * 64;
            const uint64_t o = ((uint64_t)lane_xor<STRIDE>((uint32_t)(v[j] >> 32)) << 32) | lane_xor<STRIDE>((uint32_t)v[j]);
            const bool keep_max = ((i & STRIDE) == 0) == ((i & SIZE) == 0);
            v[j] = ((v[j] > o) == keep_max) ? v[j] : o;
        }
    }
    if constexpr (STRIDE > 1) bitonic_sort<MTOP, SIZE, STRIDE / 2>(v, sort_buf, base);
    else if constexpr (SIZE < MTOP * 1024) bitonic_sort<MTOP, SIZE * 2, SIZE>(v, sort_buf, base);
}

// Maximum / sum over a wave by DPP moves; lane 63 holds the result (lanes without a source keep their own).
__device__ __forceinline__ uint32_t wave_max_last(uint32_t v) {
#define CUSA_STEP(CTRL, ROWS) { const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xF, false); v = o > v ? o : v; }
    CUSA_STEP(0x111, 0xF) CUSA_STEP(0x112, 0xF) CUSA_STEP(0x114, 0xF) CUSA_STEP(0x118, 0xF) CUSA_STEP(0x142, 0xA) CUSA_STEP(0x143, 0xC)
#undef CUSA_STEP
    return v;
}
__device__ __forceinline__ float wave_sum_last(float v) {
#define CUSA_STEP(CTRL, ROWS) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, false));
    CUSA_STEP(0x111, 0xF) CUSA_STEP(0x112, 0xF) CUSA_STEP(0x114, 0xF) CUSA_STEP(0x118, 0xF) CUSA_STEP(0x142, 0xA) CUSA_STEP(0x143, 0xC)
#undef CUSA_STEP
    return v;
}
// Maximum over the sixteen values of a 16-lane row, in every lane.
__device__ __forceinline__ uint32_t row_max16(uint32_t v) {
#define CUSA_STEP(CTRL) { const uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true); v = o > v ? o : v; }
    CUSA_STEP(0x128) CUSA_STEP(0x124) CUSA_STEP(0x122) CUSA_STEP(0x121)   // row_ror:8, 4, 2, 1
#undef CUSA_STEP
    return v;
}

// LDS words of the ranking, besides the bins and the segments.
struct RankScratch {
    float excess;                // cleared by the caller, like walk
    int walk, wave[SEL_WAVES];
};
constexpr int RANK_BINS = 2048;
enum { RANK_DONE = 0, RANK_FAILED = 1, RANK_CROWDED = 2 };

// Ranks the m <= 64 CHUNKS composites of a segment that starts at rank 0, the workgroup together: every wave holds all
// of them, 64 to a register, and compares its sixteenth of them with 64 at a time.
template <int CHUNKS>
__device__ __forceinline__ void rank_together(const uint64_t* seg, int m, int k_out, int32_t* __restrict__ out, int H) {
    const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
    uint64_t r[CHUNKS];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) r[c] = c * 64 + lane < m ? seg[c * 64 + lane] : 0;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        for (int l = w; l < 64 && c * 64 + l < m; l += SEL_WAVES) {
            const uint64_t cv = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(r[c] >> 32), l) << 32) |
                                (uint32_t)__builtin_amdgcn_readlane((int)r[c], l);
            int rank = 0;
#pragma unroll
            for (int q = 0; q < CHUNKS; ++q) rank += __popcll(__ballot(r[q] > cv));
            if (lane == 0 && rank < k_out) out[(int64_t)rank * H] = (int32_t)~(uint32_t)cv;
        }
    }
}

// Ranks the n composites mine(0) .. mine(NPT - 1) of every thread (zero: none; all at or above the score s_lo)
// and writes the picks ranked below k_out <= n, rank-major (out[rank * H]) -- without a sorting network:
// 2048 bins divide the score range evenly by value (monotone in the key, so bins are in rank order), a
// counting sort puts every composite into its bin's segment, and inside a segment -- a few entries,
// unless scores repeat -- a composite's rank is the number of entries that beat it.  The range is
// [s_lo, s_lo + 6 x the mean excess over s_lo], not up to the best score: a few very large scores
// (attention sinks, hot tokens) would otherwise stretch the bins over empty space and crowd the
// rest; whatever lies above shares the first bin.  About a fifth of the instructions of a sorting network.
// Otherwise nothing is written and the caller ranks another way: RANK_FAILED, the scores are not finite; RANK_CROWDED, they
// are, but all alike, or repeat so often that walking their segments (the sum of the squares of their lengths; WALK_MAX) would
// take longer than the network, which adds 17 us: 32 rows of 32256, k 1536, whose scores come 32 at a time 16.1 us, 126 at a
// time 24.8, 252 at a time 44.8, all different 13.3.
// seg: room for n composites; rbin: RANK_BINS zeros; *rs cleared; all
// visible to the workgroup (one barrier since).  Called by the whole workgroup.
//
// Sixteen waves on one CU: an instruction that all of them execute costs sixteen cycles, a barrier a few
// hundred, so sums and scans go by DPP and the barriers wait for LDS only.
template <int NPT, typename Mine>
__device__ __forceinline__ int rank_entries(Mine mine, int n, float s_lo, int k_out, uint64_t* seg, int* rbin,
                                            RankScratch* rs, int32_t* __restrict__ out, int H) {
    constexpr int RMAX = 32, RMAX_FIRST = 512, WALK_MAX = 1 << 18;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(wave_id());
    {
        float excess = 0.0f;
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (mine(j) != 0) excess += key_score((uint32_t)(mine(j) >> 32)) - s_lo;
        excess = wave_sum_last(excess);
        if (lane_id() == 63) atomicAdd(&rs->excess, excess);
    }
    lds_barrier();
    const float range = 6.0f * rs->excess / (float)n;    // workgroup-uniform, like all that follows
    if (!(fabsf(range) < 3.0e38f)) return RANK_FAILED;
    if (!(range > 0.0f)) return RANK_CROWDED;
    const float scale = (float)(RANK_BINS - 1) / range;
    auto bin_of = [&](uint64_t cv) {                     // bin 0 holds the best scores
        const int up = (int)((key_score((uint32_t)(cv >> 32)) - s_lo) * scale);
        return RANK_BINS - 1 - (up < 0 ? 0 : up > RANK_BINS - 1 ? RANK_BINS - 1 : up);
    };
    uint32_t slot[NPT];                                  // bin << 16 | place in the bin
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
        if (mine(j) != 0) {
            const int bn = bin_of(mine(j));
            slot[j] = ((uint32_t)bn << 16) | (uint32_t)atomicAdd(&rbin[bn], 1);
        }
    }
    lds_barrier();
    {   // counts -> first indices (thread i owns bins 2i, 2i + 1)
        const int c0 = rbin[2 * tid], c1 = rbin[2 * tid + 1];
        const int inc = wave_scan_incl(c0 + c1);
        if (lane_id() == 63) rs->wave[w] = inc;
        lds_barrier();
        int first = inc - c0 - c1;
#pragma unroll
        for (int i = 0; i < SEL_WAVES; ++i) first += i < w ? rs->wave[i] : 0;
        // only segments that reach into the wanted ranks are walked: the others may be crowded
        int walk = first + c0 < k_out && c1 > RMAX ? c1 * c1 : 0;
        if (tid == 0) walk += c0 > RMAX_FIRST ? WALK_MAX + 1 : 0;
        else if (first < k_out && c0 > RMAX) walk += c0 * c0;
        if (walk != 0) atomicAdd(&rs->walk, walk);
        rbin[2 * tid] = first;
        rbin[2 * tid + 1] = first + c0;
    }
    lds_barrier();
    if (rs->walk > WALK_MAX) return RANK_CROWDED;
#pragma unroll
    for (int j = 0; j < NPT; ++j)
        if (mine(j) != 0) seg[rbin[slot[j] >> 16] + (int)(slot[j] & 0xffffu)] = mine(j);
    lds_barrier();
    // The first bin holds whatever lies above the range (hot tokens, often with equal scores): when there are many, the
    // waves rank them together, an entry against 64 others per compare.
    const int m0 = __builtin_amdgcn_readfirstlane(rbin[1]);
    const bool many = m0 > 16;
    if (many) {
        if (m0 <= 64) rank_together<1>(seg, m0, k_out, out, H);
        else if (m0 <= 128) rank_together<2>(seg, m0, k_out, out, H);
        else if (m0 <= 256) rank_together<4>(seg, m0, k_out, out, H);
        else rank_together<RMAX_FIRST / 64>(seg, m0, k_out, out, H);
    }
    // the composites ranked below k_out lie in the segments' first k_out entries or just behind them
    for (int i = (many ? m0 : 0) + tid; i < n; i += SEL_THREADS) {
        const uint64_t cv = seg[i];
        const int bn = bin_of(cv), lo = rbin[bn], hi = bn == RANK_BINS - 1 ? n : rbin[bn + 1];
        if (lo >= k_out) break;                          // (segments are in rank order: nothing wanted from here on)
        int rank = lo;
        for (int q = lo; q < hi; q += 4) {               // four at a time: the reads overlap
            uint64_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = seg[min(q + e, hi - 1)];
#pragma unroll
            for (int e = 0; e < 4; ++e) rank += (q + e < hi && o[e] > cv) ? 1 : 0;
        }
        if (rank < k_out) out[(int64_t)rank * H] = (int32_t)~(uint32_t)cv;
    }
    return RANK_DONE;
}

// Candidates of a row that the fast path may keep, whichever wave or slice they come from.
__host__ __device__ constexpr int fast_list_cap(int mtop) { return mtop <= 2 ? 4096 : mtop <= 4 ? 7168 : 14336; }
constexpr int FAST_SAMPLE = 4;                          // sampled keys per thread
constexpr float FAST_Z = 4.0f;

// A threshold for the k_eff best of a row's N candidates from a sample of their keys: the sample is counted into
// 2048 bins that divide [lowest, highest sampled score] evenly by value, and the threshold is the lower edge of the bin
// below the one that holds the j-th largest of the sample.  Where all candidates are sampled, j = k_eff makes it a
// bound that at least k_eff candidates reach; otherwise j = f n_s + FAST_Z sqrt(f (1 - f) n_s) + 1 with f = k_eff / N,
// which leaves too few candidates once in 30 000 rows whose order has nothing to do with the scores.  The threshold only
// decides how long a row takes.
struct RowSample {
    int above, c_hi, c_lo, n_s;  // this thread's two bins (from the top), sampled keys in higher bins, sampled keys
    float smin, step;
};
struct SampleScratch {
    uint32_t hi[SEL_WAVES], not_lo[SEL_WAVES];
    int wave[SEL_WAVES], bin;
};
// sk: the thread's sampled keys (0: none).  shist: RANK_BINS zeros, written before the call (the first barrier in here
// makes them visible).  False (workgroup-uniform): no usable sample.
template <int S>
__device__ __forceinline__ bool sample_row(const uint32_t (&sk)[S], int* shist, SampleScratch* ss, RowSample* rs) {
    const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
    uint32_t hi = 0u, not_lo = 0u;
#pragma unroll
    for (int i = 0; i < S; ++i) {
        const uint32_t nk = sk[i] != 0u ? ~sk[i] : 0u;
        hi = sk[i] > hi ? sk[i] : hi;
        not_lo = nk > not_lo ? nk : not_lo;
    }
    hi = wave_max_last(hi);
    not_lo = wave_max_last(not_lo);
    if (lane == 63) {
        ss->hi[w] = hi;
        ss->not_lo[w] = not_lo;
    }
    lds_barrier();
    const uint32_t kmax = row_max16(ss->hi[lane & 15]), kmin = ~row_max16(ss->not_lo[lane & 15]);
    rs->smin = key_score(__builtin_amdgcn_readfirstlane(kmin));
    const float range = key_score(__builtin_amdgcn_readfirstlane(kmax)) - rs->smin;
    if (!(range > 0.0f && range < 3.0e38f)) return false;   // nothing sampled, all alike, or not finite
    rs->step = range * (1.0f / (RANK_BINS - 1));
    const float scale = (float)(RANK_BINS - 1) / range;
#pragma unroll
    for (int i = 0; i < S; ++i) {
        if (sk[i] != 0u) {
            const int bi = (int)((key_score(sk[i]) - rs->smin) * scale);
            atomicAdd(&shist[bi < 0 ? 0 : bi > RANK_BINS - 1 ? RANK_BINS - 1 : bi], 1);
        }
    }
    lds_barrier();
    rs->c_hi = shist[RANK_BINS - 1 - 2 * tid];
    rs->c_lo = shist[RANK_BINS - 2 - 2 * tid];
    const int inc = wave_scan_incl(rs->c_hi + rs->c_lo);
    if (lane == 63) ss->wave[w] = inc;
    lds_barrier();
    rs->above = inc - rs->c_hi - rs->c_lo;
    rs->n_s = 0;
#pragma unroll
    for (int i = 0; i < SEL_WAVES; ++i) {
        const int c = ss->wave[i];
        rs->above += i < w ? c : 0;
        rs->n_s += c;
    }
    return true;
}
// The threshold for the j-th largest of the sample, and the score that ranking may start its bins at (no lower
// than the sample's lowest, also where everything is kept).  One barrier.
__device__ __forceinline__ float sample_threshold(const RowSample& rs, int j, SampleScratch* ss, float* s_lo) {
    const int tid = threadIdx.x;
    if (rs.above < j && j <= rs.above + rs.c_hi + rs.c_lo) ss->bin = RANK_BINS - (j <= rs.above + rs.c_hi ? 1 : 2) - 2 * tid;
    lds_barrier();
    const int bin = __builtin_amdgcn_readfirstlane(ss->bin);
    const bool all = j >= rs.n_s || bin < 1;
    *s_lo = all ? rs.smin : rs.smin + (float)(bin - 1) * rs.step;
    return all ? -3.4e38f : *s_lo;
}
// What is no candidate (a position outside [lo, hi)) gets the score -infinity, which no threshold lets through.  (A
// candidate's own -infinity is lost with it: if it is wanted, too few are kept, and the row is ranked the general way.)
template <int N, typename Pos>
__device__ __forceinline__ void mask_scores(f32x4 (&x)[N / 4], Pos pos, int lo, int hi) {
#pragma unroll
    for (int u = 0; u < N; ++u) x[u >> 2][u & 3] = pos(u) < hi && pos(u) >= lo ? x[u >> 2][u & 3] : -INFINITY;
}
// Hands those of a batch of N scores per thread that are not below theta (a NaN is kept, too) to put(slot, score,
// position), with the slots of a list that the whole workgroup shares: one LDS atomic per wave and batch reserves them.
// The counter counts all; a batch that does not fit any more is left out, and what then is in the list is of no use.  (A
// share of the list per wave would need no atomic, but scores are correlated along the sequence: the best of them are in a
// few waves' parts of the row.)
template <int N, typename Val, typename Pos, typename Put>
__device__ __forceinline__ void list_push(Val val, Pos pos, float theta, int* counter, int cap, Put put) {
    uint64_t mask[N];
    int n = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        mask[u] = __ballot(!(val(u) < theta));
        n += __popcll(mask[u]);
    }
    if (n == 0) return;                                  // uniform
    int at = 0;
    if (lane_id() == 0) at = atomicAdd(counter, n);
    at = __builtin_amdgcn_readfirstlane(at);
    if (at + n > cap) return;                            // uniform
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if (!(val(u) < theta)) put(at + mbcnt(mask[u]), val(u), pos(u));
        at += __popcll(mask[u]);
    }
}
// An entry of an LDS list (the score as it is; made a composite when the list is read).
__device__ __forceinline__ uint64_t list_entry(float score, int t) {
    return ((uint64_t)__float_as_uint(score) << 32) | (uint32_t)~(uint32_t)t;
}
__device__ __forceinline__ uint64_t entry_composite(uint64_t e) {
    return ((uint64_t)score_key(__uint_as_float((uint32_t)(e >> 32))) << 32) | (uint32_t)e;
}
__device__ __forceinline__ int sample_rank_wanted(int k_eff, int n, int n_s, float z) {
    const float f = (float)k_eff / (float)n;
    return min((int)(f * (float)n_s + z * sqrtf(f * (1.0f - f) * (float)n_s)) + 1, n_s);
}

// First position of quad number x of a sample of TOTAL keys of a row of n positions (of a shorter row: past its end): runs of 16
// keys (64 bytes), spread evenly.  (Scores are correlated along the sequence: fewer, longer runs say less about the row.)
template <int TOTAL>
__device__ __forceinline__ int sample_quad(int x, int n) {
    const int runs = (n + 15) >> 4;
    return (runs <= TOTAL / 16 ? x >> 2 : (int)((uint32_t)(x >> 2) * (uint32_t)runs / (TOTAL / 16))) * 16 + (x & 3) * 4;
}

// Candidates of a slice of a long row that reach the row's threshold (slice_filter_kernel), for the ranking launch.
struct SliceLists {
    uint64_t* cand;              // [row][slice][cap] composites; nullptr: rows are not sliced
    int32_t* cnt;                // [row][slice]; above cap: some did not fit
    float* s_lo;                 // [row] score of the threshold
    int cap, n_slices, slice_len;
};
constexpr int SLICE_SAMPLE = 8;                         // sampled keys per thread
// Rows longer than this that one workgroup walks are sampled like sliced ones: of 4096 keys so few are among the k best that the threshold, where
// scores are correlated along the sequence, often lets more through than the list holds (selection layers, us, samples of 4096 and 8192 keys, scores
// correlated over 64 tokens, 3584 picks: 8 pairs of 131072, groups of 1, 198 and 105; of 220000, groups of 8, 336 and 192).
constexpr int LONG_ROW = 65536;
constexpr float SLICE_Z = 6.0f;                         // instead of FAST_Z: a second walk is that of a whole row by one workgroup

// ITEMS == -1 is the streamed kernel in a register-lean form (half the keys in flight, compiled for two
// resident workgroups per CU): with more rows than CUs two rows overlap on a CU, which gains more
// than the shorter batches lose; with one row per CU it is slower than the wide form, so few long rows
// keep ITEMS == 0.
//
// Few long rows (fewer rows than CUs, more than 32768 candidates) are cut into slices: rows of scores by
// slice_filter_kernel and a ranking launch (sl); rows of raw keys by this kernel, one workgroup per slice (blockIdx.z): a
// slice selects its own k best and leaves their composites, unsorted and padded with zeros, in
// parts[row][slice][k]; the k best of a row are among the k best of its slices, so a second launch (MERGE) selects
// and ranks among those n_slices * k composites instead of the row.  MERGE also ranks what a filtered pass kept.
//
// h, b: the workgroup's place among the H heads of B sequences, heads first; z: its slice.
template <int ITEMS, int MTOP, bool MERGE>
__device__ __forceinline__ void topk_row(int h, int b, const int z, const int B, const float* __restrict__ P, int64_t ldp,
                                         const int32_t* __restrict__ seq_lens, int32_t* __restrict__ rho_head, int H, int k,
                                         int budget, int window, int raw_keys, int n_sink, uint64_t* __restrict__ parts,
                                         int slice_len, int n_slices, const int32_t* __restrict__ only_rows, FilterState flt,
                                         SliceLists sl) {
    static_assert(!MERGE || ITEMS > 0, "the composites of a merge are held in registers");
    constexpr int NSORT = MTOP * SEL_THREADS;         // k <= NSORT
    constexpr int CAP = topk_list_cap(ITEMS, MTOP);
    extern __shared__ uint64_t sort_buf[];            // NSORT composites (aliases the histogram), then CAP list entries
    uint64_t* const cand = sort_buf + NSORT;
    __shared__ __attribute__((aligned(16))) int scratch[SEL_WAVES];
    __shared__ SelectState st;
    __shared__ int n_out, n_list;
    __shared__ RankScratch rank_st;
    __shared__ SampleScratch sample_st;
    int* hist = reinterpret_cast<int*>(sort_buf);     // 2048 ints = 8 KB <= NSORT * 8
    const int wv = __builtin_amdgcn_readfirstlane(wave_id());

    // Workgroups go to the 8 XCDs round-robin in launch order.  The heads of a sequence write the same
    // lines of the rank-major output (entry (j, h) next to (j, h+1)); with eight sequences or more, all
    // heads of a sequence are put on one XCD, whose L2 then merges their 4-byte stores into whole
    // lines instead of each XCD writing its own fragments of every line (c5: 104 MB written for a 13 MB
    // output before).
    {
        const int lin = h + H * b;
        if (lin < (B / 8) * 8 * H) {
            const int within = lin % (8 * H);
            b = (lin / (8 * H)) * 8 + (within & 7);
            h = within >> 3;
        }
    }
    // only_rows: the second chance of the filtered fast path ranks the flagged heads only
    if (only_rows && only_rows[(int64_t)b * H + h] == 0) return;
    const int L = seq_lens[b];
    if (L <= budget) return;
    const int Lc = L - window;
    // this workgroup's candidates: the positions [t_lo, t_hi) of the row (a slice of it), or -- MERGE --
    // the composites the slices left, or (flt.thr set) those the filtered pass kept for this head
    const bool slice = !MERGE && parts != nullptr;
    const int t_lo = slice ? z * slice_len : 0;
    const int t_hi = slice ? min(Lc, t_lo + slice_len) : Lc;
    uint64_t* const my_parts = parts + (((int64_t)b * H + h) * n_slices + (slice ? z : 0)) * k;
    // the first n_sink positions are kept in rho anyway and are no candidates (key 0, like the padding)
    const int k_eff = MERGE ? min(k, Lc - n_sink) : min(k, t_hi - max(t_lo, n_sink));
    if (slice && k_eff <= 0) {                        // nothing of the row falls into this slice
        for (int i = threadIdx.x; i < k; i += SEL_THREADS) my_parts[i] = 0;
        return;
    }
    const float* __restrict__ row = P + ((int64_t)b * H + h) * ldp;
    // raw_keys: the row already holds order-preserving uint32 keys (the aggregated ranking keys of
    // the votes / max-score readings) instead of binary32 scores
    auto key_of = [raw_keys](float v) { return raw_keys ? __float_as_uint(v) : score_key(v); };
    // Keys held in registers come in quads, 16-byte loads: quad q of wave w is its part of the 4096-key block
    // rev(q) + w (rev: bits reversed), so that the first quads of all waves are 256-key pieces from all over the row;
    // a key of each of four (where there are eight, of the first or the last four) is the row's sample.
    constexpr int QUADS = ITEMS > 4 ? ITEMS / 4 : 1;
    int my_tid = threadIdx.x;
    auto item_pos = [&](int i) {
        constexpr int LOG2 = QUADS >= 8 ? 3 : QUADS >= 4 ? 2 : QUADS >= 2 ? 1 : 0;
        const int q = i >> 2, rev = LOG2 == 0 ? 0 : (int)(__builtin_bitreverse32((uint32_t)q) >> (LOG2 == 0 ? 31 : 32 - LOG2));
        return t_lo + ((rev + wv) & (QUADS - 1)) * (4 * SEL_THREADS) + my_tid * 4 + (i & 3);
    };
    f32x4 x[!MERGE && ITEMS > 0 ? QUADS : 1];         // scores
    uint32_t keys[ITEMS > 0 ? ITEMS : 1];             // 0: no candidate
    int pos_of[MERGE ? ITEMS : 1];                     // MERGE: the positions that come with the keys
    if constexpr (MERGE) {
        int n_cand = n_slices * k;
        const uint64_t* __restrict__ src = my_parts;
        if (flt.thr) {
            const int64_t row = (int64_t)b * H + h;
            n_cand = flt.cand_cnt[row];
            // fewer than k kept: the threshold was too high and some of the k best are missing; more than
            // the list holds: some were dropped.  Either way the head is ranked the ordinary way later.
            if (flt.fail[row] != 0 || n_cand > flt.cap || n_cand < k_eff) {
                if (threadIdx.x == 0) {
                    flag_failed(flt, row);
                    atomicAdd(flt.n_failed, 1);
                }
                return;
            }
            src = flt.cand + row * flt.cap;
        }
        uint64_t mcv[ITEMS];                           // this thread's composites (zero: none)
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int sl = i * SEL_THREADS + threadIdx.x;
            const uint64_t cv = src[sl < n_cand ? sl : n_cand - 1];
            mcv[i] = sl < n_cand ? cv : 0;
        }
        // A filtered pass's candidates are few and most of them among the k best, so they are first ranked as they
        // are: all of them, of which only the ranks below k_eff are written.  If that does not work out
        // (crowded bins) they are selected and sorted like any row.
        if constexpr (ITEMS <= 8) {
            if (flt.thr) {
                int* const rbin = reinterpret_cast<int*>(sort_buf + ITEMS * SEL_THREADS);
                rbin[2 * threadIdx.x] = rbin[2 * threadIdx.x + 1] = 0;
                if (threadIdx.x == 0) {
                    rank_st.excess = 0.0f;
                    rank_st.walk = 0;
                }
                lds_barrier();
                if (rank_entries<ITEMS>([&](int j) { return mcv[j]; }, n_cand, key_score(flt.thr[(int64_t)b * H + h]), k_eff, sort_buf,
                                        rbin, &rank_st, rho_head + (int64_t)b * k * H + h, H) == RANK_DONE)
                    return;
                __syncthreads();
            }
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            keys[i] = (uint32_t)(mcv[i] >> 32);
            pos_of[i] = (int)~(uint32_t)mcv[i];
        }
    }
    // rows are padded to a multiple of 64 entries (ldp): a quad that starts below ldp stays inside its row
    auto load_row = [&]() {
#pragma unroll
        for (int q = 0; q < QUADS; ++q) x[q] = *reinterpret_cast<const f32x4*>(row + min(item_pos(4 * q), (int)ldp - 4));
        asm volatile("" : "+v"(my_tid));              // positions are made anew where they are needed, not kept in registers
    };
    if constexpr (!MERGE && ITEMS > 0) {
        if (!slice && !raw_keys) load_row();          // uniform
    }
    // Streamed rows (ITEMS <= 0) are walked in batches of SB keys per thread covering the positions
    // [t0, t0 + SB * 1024): key u of a thread is position t0 + ((u / 4) * 1024 + thread) * 4 + u % 4, so a
    // thread fetches 16 bytes at a time and a wave 1 KB per load.  Rows start 256-byte aligned and are
    // padded to a multiple of 64 entries (ldp), so a load that starts below ldp stays inside the row;
    // the others are clamped and, like everything at or past t_hi, masked (loads stay unconditional).
    // A slice starts at a multiple of 4096 positions, so its loads are aligned like the row's.
    constexpr int SB = ITEMS == -1 ? 8 : 16;
    auto stream_pos = [&](int t0, int u) { return t0 + ((u >> 2) * SEL_THREADS + (int)threadIdx.x) * 4 + (u & 3); };
    // The loads of the next batch are issued before the current one is worked on.
    auto stream_issue = [&](f32x4 (&x)[SB / 4], int t0) {
#pragma unroll
        for (int v = 0; v < SB / 4; ++v) {
            const int t = stream_pos(t0, 4 * v);
            x[v] = *reinterpret_cast<const f32x4*>(row + (t < (int)ldp ? t : (int)ldp - 4));
        }
    };
    auto stream_take = [&](const f32x4 (&x)[SB / 4], uint32_t (&kk)[SB], int t0) {
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const int t = stream_pos(t0, u);
            const uint32_t kv_ = key_of(x[u >> 2][u & 3]);
            kk[u] = (t < t_hi && t >= n_sink) ? kv_ : 0u;
        }
    };
    // f(scores of the batch, first position of the batch) for every batch of a streamed row; the same with keys
    auto stream_scores = [&](auto f) {
        f32x4 next[SB / 4];
        stream_issue(next, t_lo);
        for (int t0 = t_lo; t0 < t_hi; t0 += SB * SEL_THREADS) {
            f32x4 cur[SB / 4];
#pragma unroll
            for (int v = 0; v < SB / 4; ++v) cur[v] = next[v];
            stream_issue(next, t0 + SB * SEL_THREADS);   // past the row's end: clamped loads, never used
            __builtin_amdgcn_sched_barrier(0);
            f(cur, t0);
        }
    };
    auto stream_batches = [&](auto f) {
        f32x4 next[SB / 4];
        stream_issue(next, t_lo);
        for (int t0 = t_lo; t0 < t_hi; t0 += SB * SEL_THREADS) {
            uint32_t kk[SB];
            stream_take(next, kk, t0);
            stream_issue(next, t0 + SB * SEL_THREADS);
            __builtin_amdgcn_sched_barrier(0);
            f(kk, t0);
        }
    };
    auto scan = [&](auto f) {
        if constexpr (ITEMS > 0) {
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                f(keys[i], MERGE ? pos_of[i] : item_pos(i));
            }
        } else {
            stream_batches([&](const uint32_t (&kk)[SB], int t0) {
#pragma unroll
                for (int u = 0; u < SB; ++u) f(kk[u], stream_pos(t0, u));
            });
        }
    };

    // 1-3 for candidates delivered by scan_fn: the digits of the k_eff-th best score key
    // T (first_pass 1: its top digit is already in st), the position bound among the keys equal to T when they
    // straddle the cut (rare), and the survivors' composites compacted into sort_buf in any order.
    uint32_t sel_T = 0u;                              // the k_eff-th best score key, once this has run
    auto finish = [&](int first_pass, auto scan_fn) {
        radix_select(first_pass, k_eff, 0u, scan_fn, [](uint32_t skey, int, uint32_t* key) { *key = skey; return true; },
                     hist, scratch, &st);
        const uint32_t T = st.prefix;
        sel_T = T;
        const int need_eq = st.need, count_eq = st.count_eq;
        __syncthreads();
        uint32_t pos_bound = 0xffffffffu;              // take every tie
        if (count_eq > need_eq) {
            radix_select(0, need_eq, 0u, scan_fn,
                         [T](uint32_t skey, int t, uint32_t* key) { *key = ~(uint32_t)t; return skey == T; },
                         hist, scratch, &st);
            pos_bound = ~st.prefix;                    // need_eq-th smallest tying position
            __syncthreads();
        }
        if (threadIdx.x == 0) n_out = 0;
        __syncthreads();                               // also: histogram no longer needed
        // one reservation per wave: count this thread's survivors, scan the counts over the wave
        int mine = 0;
        scan_fn([&](uint32_t key, int t) {
            mine += (key > T || (key == T && (uint32_t)t <= pos_bound)) ? 1 : 0;
        });
        int slot = wave_reserve(mine, &n_out);
        scan_fn([&](uint32_t key, int t) {
            if (key > T || (key == T && (uint32_t)t <= pos_bound)) {
                if (slot < NSORT) sort_buf[slot] = ((uint64_t)key << 32) | (uint32_t)~(uint32_t)t;
                ++slot;
            }
        });
        __syncthreads();
    };

    int n_sort = 0;                                   // composites in sort_buf that only have to be sorted (0: not that far)
    // The fast path.  A threshold from a sample of the row lets the k_eff best and a few more candidates through;
    // the waves compact those into one LDS list, and they are ranked as they are
    // (rank_entries).  One look at every key, one compare: what the selection below pays for -- histogram atomics that
    // meet in a handful of digit bins, top candidates of every thread -- falls away.  Where many scores of the list are equal it
    // is sorted instead; the selection stands for rows that have no such list (scores that are not finite, more
    // candidates at the threshold than it holds, thresholds that let too few through) and for raw keys.
    if constexpr (!MERGE) {
        if (!slice && !raw_keys) {                    // uniform
            constexpr int FCAP = fast_list_cap(MTOP), NPT = FCAP / SEL_THREADS;
            int* const shist = reinterpret_cast<int*>(sort_buf + FCAP);
            int* const rbin = shist + RANK_BINS;
            const int tid = threadIdx.x, lane = lane_id();
            reinterpret_cast<u32x4*>(shist)[tid] = u32x4{0u, 0u, 0u, 0u};   // both areas
            if (tid == 0) {
                rank_st.excess = 0.0f;
                rank_st.walk = 0;
                n_list = 0;
            }
            uint64_t lv[NPT];                         // this thread's share of the list
            int n = 0;
            float s_lo = 0.0f;
            bool go = true;
            if constexpr (ITEMS == 0) {               // a long row whose slices have been filtered already
                if (sl.cand) {
                    const int64_t r0 = ((int64_t)b * H + h) * sl.n_slices;
                    for (int y = 0; y < sl.n_slices; ++y) n += min(sl.cnt[r0 + y], FCAP + 1);
                    go = n < k_eff || n > FCAP;
                    if (!go) {
                        s_lo = sl.s_lo[(int64_t)b * H + h];
#pragma unroll
                        for (int j = 0; j < NPT; ++j) {
                            int i = tid + j * SEL_THREADS;
                            lv[j] = 0;
                            if (i < n) {
                                int y = 0;
                                for (int c = sl.cnt[r0]; i >= c; c = sl.cnt[r0 + y]) {
                                    i -= c;
                                    ++y;
                                }
                                lv[j] = sl.cand[(r0 + y) * sl.cap + i];
                            }
                        }
                        lds_barrier();                // the cleared areas
                    }
                }
            }
            if (go) {
                auto mask_row = [&]() {               // a wave's quad is 256 positions: all of them candidates, some, or none
#pragma unroll
                    for (int q = 0; q < QUADS; ++q) {
                        const int first = __builtin_amdgcn_readfirstlane(item_pos(4 * q));
                        if (first < n_sink || first + 256 > t_hi) {
                            f32x4 (&xq)[1] = *reinterpret_cast<f32x4 (*)[1]>(&x[q]);
                            mask_scores<4>(xq, [&](int u) { return item_pos(4 * q + u); }, n_sink, t_hi);
                        }
                    }
                    asm volatile("" : "+v"(my_tid));
                };
                if constexpr (ITEMS > 0) mask_row();
                constexpr bool EXACT = ITEMS > 0 && ITEMS <= FAST_SAMPLE;
                RowSample rs;
                if constexpr (ITEMS > 0) {
                    uint32_t sk[FAST_SAMPLE];
#pragma unroll
                    for (int i = 0; i < FAST_SAMPLE; ++i) {
                        const int it = QUADS >= 4 ? 5 * i : QUADS == 2 ? (i < 2 ? 2 * i : 2 * i + 1) : i;   // (5 i: element i of quad i)
                        // of eight quads, every other lane samples the last four: no part of the row is left out
                        const float s = QUADS == 8 && (lane & 1) ? x[(it >> 2) + (QUADS == 8 ? 4 : 0)][it & 3] : x[it >> 2][it & 3];
                        sk[i] = s == -INFINITY ? 0u : score_key(s);
                    }
                    go = sample_row(sk, shist, &sample_st, &rs);
                } else {
                    auto sample_streamed = [&](auto keys_per_thread) {   // 16-byte loads
                        constexpr int S = decltype(keys_per_thread)::value;
                        f32x4 y[S / 4];
                        uint32_t sk[S];
#pragma unroll
                        for (int i = 0; i < S / 4; ++i)
                            y[i] = *reinterpret_cast<const f32x4*>(row + min(sample_quad<S * SEL_THREADS>(i * SEL_THREADS + tid, t_hi), (int)ldp - 4));
#pragma unroll
                        for (int i = 0; i < S; ++i) {
                            const int t = sample_quad<S * SEL_THREADS>((i >> 2) * SEL_THREADS + tid, t_hi) + (i & 3);
                            sk[i] = t < t_hi && t >= n_sink ? score_key(y[i >> 2][i & 3]) : 0u;
                        }
                        return sample_row(sk, shist, &sample_st, &rs);
                    };
                    if (ITEMS == -1 && t_hi > LONG_ROW) go = sample_streamed(std::integral_constant<int, SLICE_SAMPLE>());   // uniform
                    else go = sample_streamed(std::integral_constant<int, FAST_SAMPLE>());
                }
                // (slices that failed have told how many reach a threshold like the first)
                for (int attempt = ITEMS == 0 && sl.cand ? 1 : 0; go; ++attempt) {
                    int j = EXACT ? k_eff : sample_rank_wanted(k_eff, t_hi - max(t_lo, n_sink), rs.n_s, FAST_Z);
                    if (attempt == 1)                 // n were too few (too many): as many more (fewer) as should do, twice as many at most
                        j = min(min(2 * j, (int)(1.25f * (float)j * (float)k_eff * __builtin_amdgcn_rcpf((float)max(n, 1))) + 8), rs.n_s);
                    const float theta = sample_threshold(rs, j, &sample_st, &s_lo);
                    asm volatile("" : "+v"(my_tid));
                    auto put = [&](int slot, float score, int t) {
                        sort_buf[slot] = list_entry(score, t);
                    };
                    if constexpr (ITEMS > 0) {
                        constexpr int PB = ITEMS < 8 ? ITEMS : 8;
#pragma unroll
                        for (int i0 = 0; i0 < ITEMS; i0 += PB) {
                            list_push<PB>([&](int u) { return x[(i0 + u) >> 2][u & 3]; }, [&](int u) { return item_pos(i0 + u); }, theta, &n_list, FCAP, put);
                            __builtin_amdgcn_sched_barrier(0);   // a few masks at a time
                        }
                    } else {
                        stream_scores([&](f32x4 (&xs)[SB / 4], int t0) {
                            if (t0 < n_sink || t0 + SB * SEL_THREADS > t_hi) mask_scores<SB>(xs, [&](int u) { return stream_pos(t0, u); }, n_sink, t_hi);
                            list_push<SB>([&](int u) { return xs[u >> 2][u & 3]; }, [&](int u) { return stream_pos(t0, u); }, theta, &n_list, FCAP, put);
                        });
                    }
                    lds_barrier();
                    n = __builtin_amdgcn_readfirstlane(n_list);
                    if (n >= k_eff || attempt == 1) break;
                    lds_barrier();                    // everyone has read the count; try a lower threshold
                    if (tid == 0) n_list = 0;
                    if constexpr (ITEMS > 0) {        // (not kept in registers for this)
                        load_row();
                        mask_row();
                    }
                    lds_barrier();
                }
            }
            if (n >= k_eff && n <= FCAP) {            // uniform
                if (go) {
#pragma unroll
                    for (int j = 0; j < NPT; ++j) lv[j] = tid + j * SEL_THREADS < n ? entry_composite(sort_buf[tid + j * SEL_THREADS]) : 0;
                }
                const int res = rank_entries<NPT>([&](int j) { return lv[j]; }, n, s_lo, k_eff, sort_buf, rbin, &rank_st,
                                                  rho_head + (int64_t)b * k * H + h, H);
                if (res == RANK_DONE) return;
                lds_barrier();                        // the areas are used anew
                if (res == RANK_CROWDED) {            // all finite, so the k_eff best are among them
                    if (n <= NSORT) {
#pragma unroll
                        for (int j = 0; j < MTOP; ++j) sort_buf[tid + j * SEL_THREADS] = lv[j];
                        n_sort = NSORT;
                    } else {
                        finish(0, [&](auto f) {
#pragma unroll
                            for (int j = 0; j < NPT; ++j)
                                if (lv[j] != 0) f((uint32_t)(lv[j] >> 32), (int)~(uint32_t)lv[j]);
                        });
                        n_sort = k_eff;
                    }
                }
            }
            __syncthreads();                          // the areas are used anew below
        }
    }
    if (n_sort == 0) {                                // uniform
    // The general path, on keys.
    if constexpr (!MERGE && ITEMS > 0) {              // (fetched anew: kept beside what the fast path needs, the scores do not fit the registers)
        load_row();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int t = item_pos(i);
            const uint32_t kv_ = key_of(x[i >> 2][i & 3]);
            keys[i] = (t < t_hi && t >= n_sink) ? kv_ : 0u;
        }
        asm volatile("" : "+v"(my_tid));
    }
    // 0. a cheap lower bound for the k_eff-th best key.  Each thread keeps the MTOP largest of
    //    its own candidates (MTOP * 1024 >= k); the k_eff-th largest of those values cannot
    //    exceed the k_eff-th largest of all candidates, so its top digit d0 bounds the answer's
    //    from below and the first histogram pass may skip every key under d0 -- most of them,
    //    which matters because LDS histogram atomics are what this kernel is bound by.
    //    A streamed row keeps the maxima of 8 disjoint groups of the thread's candidates instead
    //    (one instruction per key): distinct candidates again, so the same argument holds, and
    //    with 8192 group maxima the bound is about as tight.
    //    The candidates a filtered pass kept (when ranking them as they are did not work out, above): no
    //    bound (d0 = 0) and no list for them.
    const bool direct = MERGE && flt.thr != nullptr;
    constexpr int MG = ITEMS > 0 ? MTOP : ITEMS == -1 ? 4 : 8;
    uint32_t d0 = 0u;
    if (!direct) {
    uint32_t top[MG];
#pragma unroll
    for (int j = 0; j < MG; ++j) top[j] = 0u;
    if constexpr (ITEMS > 0) {
        scan([&](uint32_t key, int) {
            uint32_t x = key;
#pragma unroll
            for (int j = 0; j < MTOP; ++j) {
                const uint32_t hi = top[j] > x ? top[j] : x;
                x = top[j] > x ? x : top[j];
                top[j] = hi;
            }
        });
    } else {
        stream_batches([&](const uint32_t (&kk)[SB], int) {
#pragma unroll
            for (int u = 0; u < SB; ++u) top[u % MG] = top[u % MG] > kk[u] ? top[u % MG] : kk[u];
        });
    }
    for (int i = threadIdx.x; i < 2048; i += SEL_THREADS) hist[i] = 0;
    if (threadIdx.x == 0) {
        st.prefix = 0;
        st.need = k_eff;
        st.count_eq = 0;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < MG; ++j) atomicAdd(&hist[top[j] >> 21], 1);
    __syncthreads();
    pick_digit<2048>(hist, scratch, &st, 21);
    d0 = st.prefix >> 21;
    __syncthreads();
    }
    // The top digit of T comes from one histogram pass over all candidates whose top digit is at
    // least d0.  Those are the only ones that can still matter; when they fit they are copied to
    // an LDS list and everything after this pass walks the list (a few entries per thread)
    // instead of every candidate again.
    for (int i = threadIdx.x; i < 2048; i += SEL_THREADS) hist[i] = 0;
    if (threadIdx.x == 0) {
        st.prefix = 0;
        st.need = k_eff;
        st.count_eq = 0;
        n_list = 0;
    }
    __syncthreads();
    int listable = 0;
    bool listed = false;
    if constexpr (ITEMS <= 0) {
        // one walk does both: each batch is counted into the histogram, the wave reserves list
        // slots for the batch's candidates and writes them (in arbitrary order; what is selected
        // from the list does not depend on it)
        stream_batches([&](const uint32_t (&kk)[SB], int t0) {
            int n_new = 0;
#pragma unroll
            for (int u = 0; u < SB; ++u) {
                const uint32_t dg = kk[u] >> 21;
                if (dg >= d0) {
                    atomicAdd(&hist[dg], 1);
                    ++n_new;
                }
            }
            int slot = wave_reserve(n_new, &n_list);
#pragma unroll
            for (int u = 0; u < SB; ++u) {
                if ((kk[u] >> 21) >= d0) {
                    if (slot < CAP) cand[slot] = ((uint64_t)kk[u] << 32) | (uint32_t)~(uint32_t)stream_pos(t0, u);
                    ++slot;
                }
            }
        });
        __syncthreads();
        pick_digit<2048>(hist, scratch, &st, 21);
        listed = n_list <= CAP;
    } else {
    scan([&](uint32_t key, int) {
        const uint32_t dg = key >> 21;
        if (dg >= d0) {
            atomicAdd(&hist[dg], 1);
            ++listable;
        }
    });
    __syncthreads();
    pick_digit<2048>(hist, scratch, &st, 21);
    if (CAP > 0 && !direct) {
        int slot = wave_reserve(listable, &n_list);
        __syncthreads();
        listed = n_list <= CAP;
        if (listed) {
            scan([&](uint32_t key, int t) {
                if ((key >> 21) >= d0) cand[slot++] = ((uint64_t)key << 32) | (uint32_t)~(uint32_t)t;
            });
            __syncthreads();
        }
    }
    }
    if (listed) {
        const int n = n_list;
        finish(1, [&](auto f) {
            for (int i = threadIdx.x; i < n; i += SEL_THREADS) {
                const uint64_t cv = cand[i];
                f((uint32_t)(cv >> 32), (int)~(uint32_t)cv);
            }
        });
    } else {
        finish(1, scan);
    }
    if (slice) {                                      // the slice's k best, in any order; the merge ranks
        for (int i = threadIdx.x; i < k; i += SEL_THREADS) my_parts[i] = i < k_eff ? sort_buf[i] : 0;
        return;
    }
    n_sort = k_eff;
    // 3a. The ranking as in the fast path; the network below remains for many equal scores, scores that are not finite and raw keys.
    if (!raw_keys && !direct) {                       // (ranking a filtered pass's candidates has been tried)
        uint64_t mine[MTOP];
#pragma unroll
        for (int j = 0; j < MTOP; ++j) {
            const int i = (int)threadIdx.x + j * SEL_THREADS;
            mine[j] = i < k_eff ? sort_buf[i] : 0;
        }
        int* const rbin = reinterpret_cast<int*>(sort_buf + NSORT);
        rbin[2 * threadIdx.x] = rbin[2 * threadIdx.x + 1] = 0;
        if (threadIdx.x == 0) {
            rank_st.excess = 0.0f;
            rank_st.walk = 0;
        }
        lds_barrier();
        if (rank_entries<MTOP>([&](int j) { return mine[j]; }, k_eff, key_score(sel_T), k_eff, sort_buf, rbin, &rank_st,
                               rho_head + (int64_t)b * k * H + h, H) == RANK_DONE)
            return;
    }
    }                                                 // n_sort == 0
    for (int i = n_sort + threadIdx.x; i < NSORT; i += SEL_THREADS) sort_buf[i] = 0;
    __syncthreads();
    // 3b. Bitonic network over NSORT = MTOP * 1024 composites, MTOP per thread in registers:
    // element j of thread (wave, lane) is index wave*64*MTOP + j*64 + lane.  A step with
    // stride < 64 exchanges between lanes of a wave, a stride of 64 .. 32*MTOP between the
    // thread's own registers, and only larger strides go through LDS with workgroup barriers.
    {
        const int lane = lane_id(), base = wave_id() * 64 * MTOP + lane;
        uint64_t v[MTOP];
#pragma unroll
        for (int j = 0; j < MTOP; ++j) v[j] = sort_buf[base + j * 64];
        bitonic_sort<MTOP, 2, 1>(v, sort_buf, base);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < MTOP; ++j) sort_buf[base + j * 64] = v[j];
        __syncthreads();
    }
    // 4. rank-major output
    int32_t* __restrict__ out = rho_head + (int64_t)b * k * H + h;
    for (int j = threadIdx.x; j < k_eff; j += SEL_THREADS)
        out[(int64_t)j * H] = (int32_t)~(uint32_t)sort_buf[j];
}

// Forms that leave room for a second workgroup on the CU.
constexpr bool topk_lean(int items, int mtop) { return mtop <= 4 && (items == -1 || (items > 0 && items <= 8)); }

template <int ITEMS, int MTOP, bool MERGE = false>
__global__ __launch_bounds__(SEL_THREADS, topk_lean(ITEMS, MTOP) ? 8 : 4) void topk_kernel(const float* __restrict__ P, int64_t ldp,
                                                            const int32_t* __restrict__ seq_lens,
                                                            int32_t* __restrict__ rho_head, int H, int k,
                                                            int budget, int window, int raw_keys, int n_sink,
                                                            uint64_t* __restrict__ parts, int slice_len, int n_slices,
                                                            const int32_t* __restrict__ only_rows, FilterState flt,
                                                            SliceLists sl) {
    topk_row<ITEMS, MTOP, MERGE>((int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z, (int)gridDim.y, P, ldp, seq_lens, rho_head, H, k, budget,
                                 window, raw_keys, n_sink, parts, slice_len, n_slices, only_rows, flt, sl);
}

// Few long rows: one workgroup would walk a row on one CU while most of the chip idles, so a row is cut into slices
// (blockIdx.z).  Every slice's workgroup takes the row's threshold from the same sample of the whole row (8192 keys:
// cheaper than a launch that does it once), and leaves those of its candidates that reach it in the slice's list, which
// holds as many as the row's ranking takes: where in the row they stand does not matter.
// topk_kernel<0, .> ranks the lists' entries, or -- if these are too many, too few or not finite -- the row.
__global__ __launch_bounds__(SEL_THREADS, 8) void slice_filter_kernel(const float* __restrict__ P, int64_t ldp,
                                                                       const int32_t* __restrict__ seq_lens, int H, int k,
                                                                       int budget, int window, int n_sink,
                                                                       const int32_t* __restrict__ only_rows, SliceLists sl) {
    __shared__ __attribute__((aligned(16))) int shist[RANK_BINS];
    __shared__ SampleScratch sample_st;
    __shared__ int n_list;
    const int h = blockIdx.x, b = blockIdx.y, z = blockIdx.z, tid = threadIdx.x;
    const int64_t r = (int64_t)b * H + h;
    if (only_rows && only_rows[r] == 0) return;
    const int L = seq_lens[b];
    if (L <= budget) return;
    const int Lc = L - window, n = Lc - n_sink, k_eff = min(k, n);
    shist[2 * tid] = shist[2 * tid + 1] = 0;
    if (tid == 0) n_list = 0;
    const float* __restrict__ row = P + r * ldp;
    f32x4 x[SLICE_SAMPLE / 4];
    int t_s[SLICE_SAMPLE / 4];
#pragma unroll
    for (int i = 0; i < SLICE_SAMPLE / 4; ++i) {
        t_s[i] = sample_quad<SLICE_SAMPLE * SEL_THREADS>(i * SEL_THREADS + tid, Lc);
        x[i] = *reinterpret_cast<const f32x4*>(row + min(t_s[i], (int)ldp - 4));
    }
    const int t_lo = z * sl.slice_len, t_hi = min(Lc, t_lo + sl.slice_len);
    // the slice's first keys are on their way while the sample is worked on; positions t0 + (v * 1024 + thread) * 4 + e,
    // clamped inside the row (padded to a multiple of 64 entries) and masked
    constexpr int V = 4;
    f32x4 y[V];
    auto request = [&](int t0) {
#pragma unroll
        for (int v = 0; v < V; ++v) y[v] = *reinterpret_cast<const f32x4*>(row + min(t0 + (v * SEL_THREADS + tid) * 4, (int)ldp - 4));
    };
    request(t_lo);
    uint32_t sk[SLICE_SAMPLE];
#pragma unroll
    for (int i = 0; i < SLICE_SAMPLE; ++i) {
        const int t = t_s[i / 4] + i % 4;
        sk[i] = t < Lc && t >= n_sink ? score_key(x[i / 4][i % 4]) : 0u;
    }
    RowSample rs;
    const bool ok = sample_row(sk, shist, &sample_st, &rs);
    float s_lo = 0.0f;
    float theta = INFINITY;
    if (ok) theta = sample_threshold(rs, sample_rank_wanted(k_eff, n, rs.n_s, SLICE_Z), &sample_st, &s_lo);
    if (tid == 0 && z == 0) sl.s_lo[r] = s_lo;
    uint64_t* const list = sl.cand + (r * sl.n_slices + z) * sl.cap;
    auto put = [&](int slot, float score, int t) {
        list[slot] = entry_composite(list_entry(score, t));
    };
    for (int t0 = t_lo; t0 < t_hi; t0 += V * 4 * SEL_THREADS) {
        f32x4 c[V];
#pragma unroll
        for (int v = 0; v < V; ++v) c[v] = y[v];
        request(t0 + V * 4 * SEL_THREADS);            // past the slice's end: never used
        auto pos = [&](int u) { return t0 + ((u >> 2) * SEL_THREADS + tid) * 4 + (u & 3); };
        if (t0 < n_sink || t0 + V * 4 * SEL_THREADS > t_hi) mask_scores<4 * V>(c, pos, n_sink, t_hi);
        list_push<4 * V>([&](int u) { return c[u >> 2][u & 3]; }, pos, theta, &n_list, sl.cap, put);
    }
    lds_barrier();
    if (tid == 0) sl.cnt[r * sl.n_slices + z] = ok ? n_list : sl.cap + 1;
}

// ---------------------------------------------------------------- union / rank / window
//
// One 1024-thread workgroup per sequence.  Slot s = j*H + h of the rank-major array is head h's
// rank-j pick; the historical part of rho is the set of the first K-W distinct tokens met when
// the slots are walked in order.  The set is a bitmap over the candidate positions in LDS (one bit
// per position: 16 KB for 131072 tokens).  A range of slots is added with one atomic OR per slot;
// the OR's return value tells whether the slot set its bit, so the number of new tokens in the
// range is exact even though, among slots of the range that name the same token, an arbitrary
// one sets it.
//
// One workgroup is all there is to work with, and the kernel is a chain of LDS round trips, barriers and
// instructions that sixteen waves execute on one CU (sixteen cycles each): what counts is the number of looks, of
// instructions per look, and of LDS operations waited for one by one.  (Four waves with four times the slots per
// thread were measured: ranges as fast, the emission twice as slow.)  As many slots
// as tokens are still wanted can be added without a look at what they hold: they cannot
// name more tokens than that.  The first range is of this kind; where heads mostly disagree it leaves
// a few per cent, the next one a few per cent of those.  Where heads agree, a range is as long as the share of
// new tokens in the last one lets expect; should it pass K-W all the same, the bits it set are cleared
// and a shorter one is taken.  The last tokens are found by a single wave in groups of 64 slots, four groups
// at a time (LDS operations of a wave are carried out in order, so each group's count is exact); the
// groups from the crossing one on are taken back, and in that one a lane's pick counts if no lower
// lane names the same token.  What is left set is the answer; it is emitted in ascending position
// order, followed by the window {L-W .. L-1}.
//
// In a selection layer the launch also carries the merge of the layer's attention partials (reduce_row,
// four rows to a workgroup, behind the B union workgroups): the union keeps B compute units
// busy and waits for LDS most of the time, and a launch of its own for the merge costs 3-5 us.
// Measured (kernel trace, union + merge before -> one launch): B1 L4096 K1024 8.4 + 2.9 -> 6.2 us, B1 L32768
// K2048 10.1 + 4.8 -> 8.0, B8 L16384 K4096 14.0 + 5.0 -> 12.4, B1 H64 L131072 K4096 13.4 + 5.8 -> 11.6.

// Adds the sink positions 0 .. n_sink-1 (never picked: they are no candidates) to the set in
// `bits` and writes the set's positions in ascending order, at most `limit` of them.  Thread i
// owns the words [i * wpt, i * wpt + wpt).  Returns n_sink.
__device__ __forceinline__ int emit_sinks_and_set(uint32_t* bits, int n_words, int n_sink, int limit, int* scratch,
                                                  int32_t* __restrict__ out) {
    const int tid = threadIdx.x;
    for (int t = tid; t < n_sink; t += SEL_THREADS) atomicOr(&bits[t >> 5], 1u << (t & 31));
    if (n_sink > 0) lds_barrier();
    const int wpt = (n_words + SEL_THREADS - 1) / SEL_THREADS;
    const int w_lo = tid * wpt, w_hi = (w_lo + wpt < n_words) ? w_lo + wpt : n_words;
    int mine = 0;
    for (int i = w_lo; i < w_hi; ++i) mine += __popc(bits[i]);
    int total;
    int off = block_scan_excl(mine, scratch, &total);
    for (int i = w_lo; i < w_hi; ++i) {
        uint32_t word = bits[i];
        while (word) {
            const int bpos = __ffs(word) - 1;
            if (off < limit) out[off] = i * 32 + bpos;
            ++off;
            word &= word - 1;
        }
    }
    return n_sink;
}

constexpr int UNION_THREADS = 1024;
constexpr int UNION_WAVES = UNION_THREADS / 64;
constexpr int UNION_RUNS = 4;                         // runs of UNION_THREADS slots held in registers at a time
constexpr int UNION_MAX_POSITIONS = 144 * 1024 * 8;   // candidate positions a 144 KB bitmap covers

// What the merge of split-K partials needs (attn_reduce_kernel, and the union launch of a selection layer).
struct ReduceArgs {
    const float* part_acc;       // [row][stride_splits][128]; row = sequence * H + head
    const float* part_ml;        // [row][stride_splits][2]
    uint16_t* out;               // [row][128]
    const int32_t* n_tok;        // [B] tokens of the list a sequence attended to (clipped to n_clip)
    int n_clip, stride_splits, chunk;
    float* lse;                  // optional
    int rows;                    // B * H
};
constexpr int REDUCE_THREADS = 256;                   // threads per row
constexpr int UNION_REDUCE_ROWS = UNION_THREADS / REDUCE_THREADS;
constexpr int UNION_IDLE_WORDS = 64;
constexpr int UNION_CLAIMS = 1024;                    // entries of each of two claim tables
constexpr int UNION_WALK = 1024;                      // slots a single wave walks at most before the workgroup looks again
struct ReduceLds {
    float a[8][D];
    float m[8], l[8];
};
template <bool ALONE>
__device__ __forceinline__ void reduce_row(const ReduceArgs& r, int row, int seq, int tid, ReduceLds& lds);

__global__ __launch_bounds__(UNION_THREADS) void union_kernel(const int32_t* __restrict__ rho_head,
                                                             const int32_t* __restrict__ seq_lens,
                                                             int32_t* __restrict__ idx, int32_t* __restrict__ cnt,
                                                             int B, int H, int k, int budget, int window, int n_sink,
                                                             ReduceArgs red) {
    // 64 words where lanes with nothing to add send their atomic, then the set: ceil(Lc / 32) words; merging
    // workgroups: a ReduceLds
    extern __shared__ __attribute__((aligned(16))) uint32_t union_lds[];
    uint32_t* const bits = union_lds + UNION_IDLE_WORDS;
    __shared__ int wave_cnt[2 * UNION_WAVES];
    __shared__ int scratch[UNION_WAVES];
    __shared__ int picks[UNION_WALK];                 // the picks of a 1024-slot range, by slot
    __shared__ uint32_t claims[2 * UNION_CLAIMS];         // lane << 24 | token: who names it first in the crossing group
    __shared__ int walk_cum;
    const int b = blockIdx.x, tid = threadIdx.x, lane = lane_id(), w = wave_id();
    if (b >= B) {                                     // the attention partials of a (sequence, head) row
        const int sub = __builtin_amdgcn_readfirstlane(tid / REDUCE_THREADS);
        const int row = (b - B) * UNION_REDUCE_ROWS + sub;
        reduce_row<false>(red, row, min(row, red.rows - 1) / H, tid % REDUCE_THREADS, reinterpret_cast<ReduceLds*>(union_lds)[sub]);
        return;
    }
    const int32_t* __restrict__ rho = rho_head + (int64_t)b * k * H;
    int raw[UNION_RUNS];                              // picks on their way (below); the first are asked for before the length is here
    auto request_picks = [&](int s0) {
#pragma unroll
        for (int u = 0; u < UNION_RUNS; ++u) raw[u] = rho[min(s0 + u * UNION_THREADS + tid, k * H - 1)];
    };
    request_picks(0);
    const int L = seq_lens[b];
    int32_t* __restrict__ out = idx + (int64_t)b * budget;
    if (L <= budget) {
        for (int t = tid; t < L; t += UNION_THREADS) out[t] = t;
        if (tid == 0) cnt[b] = L;
        return;
    }
    const int Lc = L - window;
    const int k_eff = k < Lc - n_sink ? k : Lc - n_sink;
    const int S = k_eff * H;
    const int n_hist = budget - window - n_sink;      // picks to keep; the sink positions come on top
    const int n_words = (Lc + 31) >> 5;

    // The slots are looked at through a window of UNION_RUNS * 1024 slots held in registers: tok[u] of thread i is
    // slot win + u * 1024 + i (-1: past the end; a pick is always a candidate position).  The next window's picks
    // are requested early, with clamped, unconditional loads; the empty asm keeps the compiler from turning
    // them into one branch each.
    constexpr int WINDOW = UNION_RUNS * UNION_THREADS;
    int tok[UNION_RUNS];
    auto take_picks = [&](int s0) {
#pragma unroll
        for (int u = 0; u < UNION_RUNS; ++u) asm volatile("" : "+v"(raw[u]));
#pragma unroll
        for (int u = 0; u < UNION_RUNS; ++u) tok[u] = (s0 + u * UNION_THREADS + tid < S && (uint32_t)raw[u] < (uint32_t)Lc) ? raw[u] : -1;
    };
    for (int i = tid; i < n_words; i += UNION_THREADS) bits[i] = 0u;
    for (int i = tid; i < 2 * UNION_CLAIMS; i += UNION_THREADS) claims[i] = 64u << 24;
    lds_barrier();
    // workgroup total of per-wave counts (wave-uniform argument); wave_cnt alternates between two
    // halves so that one barrier per call is enough
    int parity = 0;
    auto block_total = [&](int wave_total) {
        int* const slot = wave_cnt + parity * UNION_WAVES;
        parity ^= 1;
        if (lane == 0) slot[w] = wave_total;
        lds_barrier();
        int v = slot[lane & (UNION_WAVES - 1)];
        v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);   // row_ror:8, 4, 2, 1: the sum over the row
        v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, true);
        v += __builtin_amdgcn_update_dpp(0, v, 0x122, 0xF, 0xF, true);
        v += __builtin_amdgcn_update_dpp(0, v, 0x121, 0xF, 0xF, true);
        return __builtin_amdgcn_readfirstlane(v);
    };
    // adds the lanes' tokens (-1: none); the bit a lane set, or 0
    auto add_to_set = [&](int t) -> uint32_t {
        const uint32_t bit = t >= 0 ? 1u << (t & 31) : 0u;
        const uint32_t old = atomicOr(&union_lds[t >= 0 ? UNION_IDLE_WORDS + (t >> 5) : lane], bit);
        return bit & ~old;
    };
    constexpr float WALK_SLOTS = 384.0f;               // expected rest that a single wave walks
    int cum = 0;                                       // distinct tokens in the set
    float slots_per_new = 1.0f;                        // of the last range
    int win = 0, lo = 0;                               // the window's first slot; its slots taken so far
    take_picks(0);
    request_picks(WINDOW);
    while (cum < n_hist && win + lo < S) {             // uniform
        if (lo >= WINDOW) {
            win += WINDOW;
            lo = 0;
            take_picks(win);
            request_picks(win + WINDOW);
        }
        const int rem = n_hist - cum;
        const float expect = (float)rem * slots_per_new;
        if (expect > WALK_SLOTS || lo == 0) {
            int len = min(max(rem, (int)(expect * 0.75f)), WINDOW - lo);
            for (;;) {                                 // shortened until it fits; at len <= rem it does
                // Neighbouring slots are neighbouring heads at one rank and often name the same token; a lane whose
                // left neighbour in its 16-lane row has the same pick leaves the atomic to it (same-address LDS
                // atomics of one instruction are carried out one after the other; for the same reason lanes that
                // stay out add zero to a word of their own).  Where a range starts inside a row, its first lane's
                // neighbour is out of the range and does not count.
                uint32_t got[UNION_RUNS];
#pragma unroll
                for (int u = 0; u < UNION_RUNS; ++u) {
                    const int mine = (uint32_t)(u * UNION_THREADS + tid - lo) < (uint32_t)len ? tok[u] : -1;
                    const int left = __builtin_amdgcn_update_dpp(-2, mine, 0x111, 0xF, 0xF, false);   // row_shr:1; -2 into lane 0 of a row
                    got[u] = add_to_set(mine != left ? mine : -1);
                }
                int wave_added = 0;
#pragma unroll
                for (int u = 0; u < UNION_RUNS; ++u) wave_added += __popcll(__ballot(got[u] != 0u));
                const int added = block_total(wave_added);
                if (cum + added <= n_hist) {
                    cum += added;
                    lo += len;
                    slots_per_new = (float)len * __builtin_amdgcn_rcpf((float)max(added, 1));
                    break;
                }
                // too far (only where len > rem): take the range back; the rest is expected in its first part
#pragma unroll
                for (int u = 0; u < UNION_RUNS; ++u)
                    if (got[u]) atomicAnd(&bits[tok[u] >> 5], ~got[u]);
                len = min(max(rem, (int)((float)(len * 7 / 8) * (float)rem * __builtin_amdgcn_rcpf((float)added))), len - 1);
                lds_barrier();
            }
            continue;
        }
        // one wave walks the next slots of the window, at most UNION_WALK
        const int hi = min(lo + UNION_WALK, WINDOW);
#pragma unroll
        for (int u = 0; u < UNION_RUNS; ++u) {
            const int at = u * UNION_THREADS + tid - lo;
            if ((uint32_t)at < (uint32_t)UNION_WALK) picks[at] = tok[u];
        }
        lds_barrier();
        if (w == 0) {                                  // its LDS accesses happen in program order
            int c_all = cum;
            for (int g0 = 0; g0 * 64 < hi - lo && c_all < n_hist; g0 += 4) {
                int g_tok[4], c[4];
                uint32_t g_won[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) g_tok[g] = (g0 + g) * 64 + lane < hi - lo ? picks[(g0 + g) * 64 + lane] : -1;
#pragma unroll
                for (int g = 0; g < 4; ++g) g_won[g] = add_to_set(g_tok[g]);
                int run = c_all, gx = 0;               // the group in which K-W is reached; 4: none
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    c[g] = __popcll(__ballot(g_won[g] != 0u));
                    run += c[g];
                    gx += run < n_hist ? 1 : 0;
                }
                int t = -1;                            // the lane's pick in that group
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    c_all += g < gx ? c[g] : 0;
                    t = g == gx ? g_tok[g] : t;
                    if (g >= gx && g_won[g]) atomicAnd(&bits[g_tok[g] >> 5], ~g_won[g]);   // taken back
                }
                if (gx < 4) {
                    // A pick of the crossing group counts only if no lower lane names its token.  The lanes
                    // claim an entry for their token, the lowest lane keeps it; an entry kept for another token
                    // leaves the question open (for all lanes with that token), which a second entry answers, or
                    // (rarely) a comparison of all lanes.
                    const uint32_t bit = t >= 0 ? 1u << (t & 31) : 0u;
                    const bool fresh = t >= 0 && !(bits[t >= 0 ? t >> 5 : 0] & bit);
                    const uint32_t claim = ((uint32_t)lane << 24) | (uint32_t)(t & 0xffffff);
                    bool open = fresh, dup = false;
#pragma unroll
                    for (int round = 0; round < 2; ++round) {
                        uint32_t* const entry = &claims[round == 0 ? t & (UNION_CLAIMS - 1) : UNION_CLAIMS + (((uint32_t)t * 2654435761u) >> 22)];
                        if (open) {
                            atomicMin(entry, claim);
                            const uint32_t kept = *entry;
                            open = ((kept ^ claim) & 0xffffffu) != 0u;
                            dup = !open && kept != claim;
                        }
                    }
                    if (__ballot(open)) {
                        for (int l = 0; l < 63; ++l) {
                            const int tl = __builtin_amdgcn_readlane(t, l);
                            dup |= (l < lane) && (tl == t);
                        }
                    }
                    const bool is_new = fresh && !dup;
                    const uint64_t ballot = __ballot(is_new);
                    if (is_new && c_all + mbcnt(ballot) < n_hist) atomicOr(&bits[t >> 5], bit);
                    c_all = n_hist;
                }
            }
            if (lane == 0) walk_cum = c_all;
        }
        lds_barrier();
        const int now = __builtin_amdgcn_readfirstlane(walk_cum);
        slots_per_new = (float)(hi - lo) * __builtin_amdgcn_rcpf((float)max(now - cum, 1));
        cum = now;
        lo = hi;
    }
    int n_take = cum;                                  // n_hist, or fewer distinct picks in total (k < K-W only)
    n_take += emit_sinks_and_set(bits, n_words, n_sink, n_hist + n_sink, scratch, out);
    for (int j = tid; j < window; j += UNION_THREADS) out[n_take + j] = L - window + j;
    if (tid == 0) cnt[b] = n_take + window;
}

// ---------------------------------------------------------------- filtered selection: the threshold
//
// Writing a score for every (head, cached token) is what the selection layer's pass pays most for
// beyond its reads, and the per-head top-k then walks all of them again.  The fast path of a selection
// layer writes only the scores that can matter.  A first, small launch (this kernel) scores a SAMPLE
// of the tokens -- every 16th tile of 64, fewer of a very long sequence -- and takes, per head, a
// threshold theta from the sample such that with overwhelming probability at least k and not many more than k of the head's
// candidates score >= theta; the pass then keeps only those (as (score key, position) composites,
// compacted per head) and the top-k ranks among them.  theta is only a guess, so everything that
// depends on it is checked: a head whose kept candidates turn out fewer than k (theta too high) or more
// than the buffers hold (theta too low, or many equal scores) is flagged, and the flagged heads are
// scored and ranked again the ordinary way (score_kernel and topk_kernel in their flagged-only forms).
// The result never depends on theta; only the time does.
//
// The sample of a head has n_s candidates out of n (every position in a sampled tile that is a
// candidate); with the target fraction f = k / n, theta is at or just below the j-th largest of the
// sample, where
//   j = f n_s + FILTER_Z sqrt(f (1 - f) n_s) + 1:
// the number of sample members among the head's true top k is hypergeometric with mean f n_s and
// standard deviation below sqrt(f (1 - f) n_s), so it exceeds j - 1 with probability ~ 3e-7 at
// FILTER_Z = 5 for tokens in no particular order (ordered inputs can defeat any fixed sample; they cost
// the second chance, nothing else).  A head whose expected share of kept candidates is above
// FILTER_MAX_SHARE, or whose kept candidates would likely overflow its buffer, gains nothing from the
// filter and is flagged at once.
//
// One 1024-thread workgroup per (sequence, KV head).  Every wave scores sampled tiles on its own,
// straight from memory on the matrix cores (below); the keys of the sample stay in LDS, [head][slot].  Then a quarter of the workgroup works on each
// head: the sample's scores are counted into 2048 bins that divide [lowest, highest sample score]
// evenly (by value, not by key: keys are dense where scores are small and a digit of the key would
// put most of the sample into a handful of bins), the bin that holds the j-th largest is found by a
// scan from the top, and theta is the smallest sample key in that bin -- so the number of sample
// members at or above theta is known exactly (j' >= j), and the expected share is j' / (n_s + 1).
constexpr int SAMPLE_STEP = 16;                       // every 16th tile at least ...
constexpr int SAMPLE_MAX_TILES = 64;                  // ... and 64 tiles (4096 sample slots) per sequence at most
constexpr float FILTER_Z = 5.0f;
constexpr float FILTER_MAX_SHARE = 0.4f;
constexpr int THR_BINS = 2048;

// Expected number of kept candidates plus three standard deviations, for a head with n candidates,
// n_s of them sampled, jp sample members at or above the threshold.
__host__ __device__ inline float filter_kept_bound(float n, float n_s, float jp) {
    const float share = jp / (n_s + 1.0f);
    return n * (share + 3.0f * sqrtf(share * (1.0f - share) / (n_s > 1.0f ? n_s : 1.0f)));
}
// j of the account above.
__host__ __device__ inline int filter_sample_rank(float k_eff, float n, float n_s) {
    const float frac = k_eff / n;
    return (int)(frac * n_s + FILTER_Z * sqrtf(frac * (1.0f - frac) * n_s)) + 1;
}

template <int GQ, bool PAGED>
__global__ __launch_bounds__(SEL_THREADS) void sample_threshold_kernel(const uint16_t* __restrict__ q, int H, int k,
                                                                        int budget, int window,
                                                                        int n_slots_max, FilterState f, KvView kv) {
    static_assert(GQ <= 4, "a quarter of the workgroup per head");
    extern __shared__ uint32_t thr_lds_buf[];         // keys [GQ][n_slots_max], then bins [GQ][THR_BINS]
    uint32_t* const keys_all = thr_lds_buf;
    int* const hist_all = reinterpret_cast<int*>(thr_lds_buf + GQ * n_slots_max);
    __shared__ uint32_t red_min[4][4], red_max[4][4], thr_min[4];
    __shared__ int red_cnt[4][4], wave_sum[4][4], sel_bin[4], sel_jp[4];
    const int kvh = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row0 = (int64_t)b * H + kvh * GQ;     // first head of the group
    if (tid < GQ) {
        f.cand_cnt[row0 + tid] = 0;
        f.fail[row0 + tid] = 0;
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *f.n_failed = 0;   // counted by the top-k, a later launch
    const int L = kv.seq_lens[b];
    if (L <= budget) {                                  // rho is every token: nothing is selected
        if (tid < GQ) f.thr[row0 + tid] = 0xffffffffu;
        return;
    }
    const int Lc = L - window, n = Lc - f.n_sink, k_eff = k < n ? k : n;
    const int tiles_all = (Lc + 63) >> 6;
    // every SAMPLE_STEP-th tile of this sequence, or as many tiles as the launch has LDS for (a short
    // sequence in a cache laid out for long ones is still sampled densely)
    const int max_tiles = n_slots_max >> 6;
    const int tile_step = max(SAMPLE_STEP, (tiles_all + max_tiles - 1) / max_tiles);
    const int n_tiles = (tiles_all + tile_step - 1) / tile_step;
    const int n_slots = n_tiles * 64;

    // The sample's scores come from V_MFMA_F32_16X16X16_BF16, 16 tokens x 16 heads (GQ of them real) per
    // instruction: lane l holds, of token l % 16 and of head l % 16, the 16-byte chunks (4 j + l / 16) of
    // the 128 columns, j = 0 .. 3 -- the order in which columns are summed does not matter here, a sample
    // score only helps to guess a threshold and need not be the score the pass computes to the last bit.
    // A load instruction reads 64 contiguous bytes of each of 16 rows.
    const int m16 = lane & 15, kg = lane >> 4;
    u32x4 qreg[4];
#pragma unroll
    for (int jc = 0; jc < 4; ++jc) {
        qreg[jc] = u32x4{0u, 0u, 0u, 0u};
        if (m16 < GQ) qreg[jc] = *reinterpret_cast<const u32x4*>(q + (row0 + m16) * D + (jc * 4 + kg) * 8);
    }
    for (int s = wave; s < n_tiles; s += SEL_WAVES) {
        const int t0 = s * tile_step * 64;
#pragma unroll
        for (int pair = 0; pair < 2; ++pair) {
            u32x4 stage[2][4];
#pragma unroll
            for (int g2 = 0; g2 < 2; ++g2) {
                const int t = t0 + (pair * 2 + g2) * 16 + m16;
                const uint16_t* __restrict__ krow = kv.k + row_offset<PAGED>(kv, b, kvh, min(t, Lc - 1));
#pragma unroll
                // (plain loads: the sampled tiles are read again by the pass, from the last-level cache if still there)
                for (int jc = 0; jc < 4; ++jc) stage[g2][jc] = *reinterpret_cast<const u32x4*>(krow + (jc * 4 + kg) * 8);
            }
#pragma unroll
            for (int g2 = 0; g2 < 2; ++g2) {
                f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int jc = 0; jc < 4; ++jc) {
                    const s16x4 a_lo = __builtin_bit_cast(s16x4, make_uint2(stage[g2][jc].x, stage[g2][jc].y));
                    const s16x4 a_hi = __builtin_bit_cast(s16x4, make_uint2(stage[g2][jc].z, stage[g2][jc].w));
                    const s16x4 b_lo = __builtin_bit_cast(s16x4, make_uint2(qreg[jc].x, qreg[jc].y));
                    const s16x4 b_hi = __builtin_bit_cast(s16x4, make_uint2(qreg[jc].z, qreg[jc].w));
                    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a_lo, b_lo, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a_hi, b_hi, acc, 0, 0, 0);
                }
                // the lane holds, for head l % 16, the tokens 4 (l / 16) + i of this group of 16
                if (m16 < GQ) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int m = (pair * 2 + g2) * 16 + kg * 4 + i, t = t0 + m;
                        const bool valid = t < Lc && t >= f.n_sink;   // key 0 for what is no candidate
                        keys_all[m16 * n_slots_max + s * 64 + m] = valid ? score_key(acc[i]) : 0u;
                    }
                }
            }
        }
    }
    __syncthreads();

    // a quarter of the workgroup (4 waves) per head; quarters without a head only keep the barriers company
    const int hq = tid >> 8, tq = tid & 255, wq = tq >> 6;
    const bool has_head = hq < GQ;
    const uint32_t* const keys = keys_all + (has_head ? hq : 0) * n_slots_max;
    int* const hist = hist_all + (has_head ? hq : 0) * THR_BINS;
    {
        int cnt = 0;
        uint32_t lo = 0xffffffffu, hi = 0u;
        if (has_head) {
            for (int sl = tq; sl < n_slots; sl += 256) {
                const uint32_t key = keys[sl];
                if (key != 0u) {
                    ++cnt;
                    lo = key < lo ? key : lo;
                    hi = key > hi ? key : hi;
                }
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            cnt += __shfl_xor(cnt, o);
            const uint32_t lo2 = __shfl_xor(lo, o), hi2 = __shfl_xor(hi, o);
            lo = lo2 < lo ? lo2 : lo;
            hi = hi2 > hi ? hi2 : hi;
        }
        if (lane == 0) {
            red_cnt[hq][wq] = cnt;
            red_min[hq][wq] = lo;
            red_max[hq][wq] = hi;
        }
        for (int i = tq; i < THR_BINS; i += 256) hist[i] = 0;
        if (tq == 0) thr_min[hq] = 0xffffffffu;
    }
    __syncthreads();
    int n_s = 0;
    uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        n_s += red_cnt[hq][w];
        kmin = red_min[hq][w] < kmin ? red_min[hq][w] : kmin;
        kmax = red_max[hq][w] > kmax ? red_max[hq][w] : kmax;
    }
    const int j = filter_sample_rank((float)k_eff, (float)n, (float)n_s);
    const float smin = key_score(kmin), range = key_score(kmax) - smin;
    // no usable guess: too few in the sample, or scores that are not finite or all alike
    bool bad = !has_head || j >= n_s || !(range > 0.0f && range < 3.0e38f);
    const float scale = bad ? 0.0f : (float)(THR_BINS - 1) / range;
    auto bin_of = [&](uint32_t key) {
        const int bi = (int)((key_score(key) - smin) * scale);
        return bi < 0 ? 0 : bi > THR_BINS - 1 ? THR_BINS - 1 : bi;
    };
    if (!bad) {
        for (int sl = tq; sl < n_slots; sl += 256) {
            const uint32_t key = keys[sl];
            if (key != 0u) atomicAdd(&hist[bin_of(key)], 1);
        }
    }
    __syncthreads();
    {   // thread i of the quarter owns the 8 bins [2048 - 8 (i + 1), 2048 - 8 i), walked from the top
        int local[8], sum = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            local[u] = hist[THR_BINS - 1 - (tq * 8 + u)];
            sum += local[u];
        }
        int inc = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(inc, o);
            if (lane >= o) inc += up;
        }
        if (lane == 63) wave_sum[hq][wq] = inc;
        __syncthreads();
        int above = inc - sum;                          // sample members in higher bins, owned by lower threads
        for (int w = 0; w < wq; ++w) above += wave_sum[hq][w];
        if (!bad && above < j && j <= above + sum) {
            int run = above;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (run < j && j <= run + local[u]) {
                    sel_bin[hq] = THR_BINS - 1 - (tq * 8 + u);
                    sel_jp[hq] = run + local[u];
                }
                run += local[u];
            }
        }
    }
    __syncthreads();
    if (!bad) {
        const int bsel = sel_bin[hq];
        uint32_t lo = 0xffffffffu;
        for (int sl = tq; sl < n_slots; sl += 256) {
            const uint32_t key = keys[sl];
            if (key != 0u && bin_of(key) == bsel) lo = key < lo ? key : lo;
        }
        if (lo != 0xffffffffu) atomicMin(&thr_min[hq], lo);
    }
    __syncthreads();
    if (has_head && tq == 0) {
        const int64_t row = row0 + hq;
        if (!bad) {
            const float jp = (float)sel_jp[hq];
            bad = jp / (float)(n_s + 1) > FILTER_MAX_SHARE || filter_kept_bound((float)n, (float)n_s, jp) > (float)f.cap;
        }
        f.thr[row] = bad ? 0xffffffffu : thr_min[hq];
        if (bad) flag_failed(f, row);
    }
}

// Aggregation for the other two readings of "globally ranked" (Sec. 3.2 names no ranking key):
// one key per candidate position, larger = better, 0 = proposed by no head.
//   votes     : (number of proposing heads) << 13 | (8191 - best rank among them)
//   max score : score_key of the largest score among the proposing heads
// The unified list is then the top K-W positions by (key descending, position ascending), which the
// per-head top-k kernel computes from the key row (raw_keys).  One workgroup per sequence walks
// the H * k_eff picks; key rows live in the workspace: agg[b][0][.] keys, agg[b][1][.] best ranks.
constexpr int RANK_VOTES_SHIFT = 13;                  // ranks are below 8192

__global__ __launch_bounds__(SEL_THREADS) void rank_aggregate_kernel(const int32_t* __restrict__ rho_head,
                                                                      const float* __restrict__ P, int64_t ldp,
                                                                      const int32_t* __restrict__ seq_lens,
                                                                      uint32_t* __restrict__ agg, int64_t ld_agg, int H,
                                                                      int k, int budget, int window, int by_score,
                                                                      int n_sink) {
    const int b = blockIdx.x, tid = threadIdx.x;
    const int L = seq_lens[b];
    if (L <= budget) return;
    const int Lc = L - window;
    const int k_eff = k < Lc - n_sink ? k : Lc - n_sink;
    const int S = k_eff * H;
    uint32_t* const key = agg + (int64_t)b * 2 * ld_agg;
    uint32_t* const best = key + ld_agg;
    for (int t = tid; t < Lc; t += SEL_THREADS) {
        key[t] = 0u;
        best[t] = 0u;
    }
    __threadfence();
    __syncthreads();
    const int32_t* __restrict__ rho = rho_head + (int64_t)b * k * H;
    for (int s = tid; s < S; s += SEL_THREADS) {
        const int j = s / H, h = s - j * H;
        const int t = rho[s];
        if ((uint32_t)t >= (uint32_t)Lc) continue;    // never: a pick is a candidate position
        if (by_score) {
            atomicMax(&key[t], score_key(P[((int64_t)b * H + h) * ldp + t]));
        } else {
            atomicAdd(&key[t], 1u << RANK_VOTES_SHIFT);
            atomicMax(&best[t], (uint32_t)(8191 - j));
        }
    }
    if (by_score) return;
    __threadfence();
    __syncthreads();
    for (int t = tid; t < Lc; t += SEL_THREADS) {
        // the atomics above were carried out in L2: read there, not in this CU's L1
        const uint32_t v = __hip_atomic_load(&key[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t r = __hip_atomic_load(&best[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v) key[t] = v | r;
    }
}

// Head-to-head selection (the per-head variant the paper compares with, Sec. 3.2 and the
// generalization figure): head h of sequence b keeps ITS OWN first K-W ranked picks plus the window.
// One workgroup per (head, sequence): the picks (distinct positions) are set in an LDS bitmap over
// the candidate positions and emitted in ascending order like the unified set.
// idx_head [B][H][budget]; cnt[b] = min(K, L_b) is the same for every head.
__global__ __launch_bounds__(SEL_THREADS) void per_head_rho_kernel(const int32_t* __restrict__ rho_head,
                                                                    const int32_t* __restrict__ seq_lens,
                                                                    int32_t* __restrict__ idx_head,
                                                                    int32_t* __restrict__ cnt, int H, int k,
                                                                    int budget, int window, int n_sink) {
    extern __shared__ uint32_t bits[];                // ceil(Lc / 32) words
    __shared__ __attribute__((aligned(16))) int scratch[SEL_WAVES];
    const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int L = seq_lens[b];
    int32_t* __restrict__ out = idx_head + ((int64_t)b * H + h) * budget;
    if (L <= budget) {
        for (int t = tid; t < L; t += SEL_THREADS) out[t] = t;
        if (tid == 0 && h == 0) cnt[b] = L;
        return;
    }
    const int Lc = L - window;
    const int k_eff = k < Lc - n_sink ? k : Lc - n_sink;
    const int n_hist = min(budget - window - n_sink, k_eff);   // = K - W - n_sink: k is at least that, and so is Lc - n_sink
    const int n_words = (Lc + 31) >> 5;
    for (int i = tid; i < n_words; i += SEL_THREADS) bits[i] = 0u;
    __syncthreads();
    const int32_t* __restrict__ rho = rho_head + (int64_t)b * k * H + h;   // rank j at rho[j * H]
    for (int j = tid; j < n_hist; j += SEL_THREADS) {
        const int t = rho[(int64_t)j * H];
        if ((uint32_t)t < (uint32_t)Lc) atomicOr(&bits[t >> 5], 1u << (t & 31));
    }
    __syncthreads();
    const int n_take = n_hist + emit_sinks_and_set(bits, n_words, n_sink, n_hist + n_sink, scratch, out);
    for (int j = tid; j < window; j += SEL_THREADS) out[n_take + j] = L - window + j;
    if (tid == 0 && h == 0) cnt[b] = n_take + window;
}

// ---------------------------------------------------------------- attention (split-K flash-decode)
//
// grid (n_splits, G, B), 256 threads.  A workgroup owns a contiguous run of the
// sequence's token list (all tokens, or rho) for one KV head; the GQ query heads of
// that group sit in LDS as bf16.  A 256-byte K or V row is read by 16 lanes with one
// 16-byte load each; a wave therefore covers 4 rows per load instruction and TI*4
// rows per iteration.  The wave parks its K rows in LDS and re-reads them one row per
// lane, which is the operand layout of the 4x4x4 bf16 MFMA: 32 instructions give every
// lane the scores of its token for four heads.  Softmax is the usual running (max, sum)
// rescale per iteration with one exp per (token, head); the numerators go back through
// LDS to the lanes that hold that token's V row, and P.V accumulates 8 columns per lane.
// The four waves are merged through LDS into one partial (m, l, acc[128]) per
// head.  With one split that is the result and is written as bf16; otherwise the
// partial goes to the workspace and attn_reduce_kernel merges the splits, or, where runs are short,
// further workgroups of the launch (wait_and_merge).  (A merge by the last workgroup to arrive was measured and is slower:
// the fence, the ticket and then its reads of the other workgroups' partials come one after the other.)

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// max over the 16 lanes of a DPP row; every lane of the row gets the result
__device__ __forceinline__ float row_max16(float v) {
    v = fmaxf(v, dpp_move<0xB1>(v));
    v = fmaxf(v, dpp_move<0x4E>(v));
    v = fmaxf(v, dpp_move<0x141>(v));
    v = fmaxf(v, dpp_move<0x140>(v));
    return v;
}

// sum over the 16 lanes of a DPP row; every lane of the row gets the result
__device__ __forceinline__ float row_sum16(float v) {
    v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_move<0x141>(v);   // row_half_mirror
    v += dpp_move<0x140>(v);   // row_mirror
    return v;
}

constexpr int ATTN_THREADS = 64 * ATTN_WAVES;

// Workgroup `split` of a (sequence, KV head) owns tokens [split*chunk, split*chunk + chunk) of
// the token list; a list of n tokens keeps ceil(n / chunk) workgroups busy (at least one) and
// the others leave at once, so short sequences of a ragged batch cost nothing.
__host__ __device__ inline int attn_active_splits(int n, int chunk) {
    const int a = (n + chunk - 1) / chunk;
    return a < 1 ? 1 : a;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// V_PERMLANE32_SWAP / V_PERMLANE16_SWAP exchange halves (rows 2,3 of a with rows 0,1 of b) or
// odd/even 16-lane rows (rows 1,3 of a with rows 0,2 of b) of two registers.  Adding the two
// results folds a and b over that lane bit at once: the lanes whose bit is 0 end up with the
// sum of a, the others with the sum of b.
__device__ __forceinline__ float fold_halves(float a, float b) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float fold_rows(float a, float b) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
// max of a lane's value and the one 16 (32) lanes away, in every lane
__device__ __forceinline__ float max_with_row_neighbour(float v) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float max_with_other_half(float v) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), lane));
}

__device__ __forceinline__ int wave_base_of(unsigned tid) { return (int)(tid >> 6); }

// ---- merge of a pair's pieces inside the attention launch
//
// Where a layer's pieces are short, the second launch that merges them costs the host as much as the first (3 us each) and the GPU the
// time between two kernels.  There the merge is done by further workgroups of the same launch, dispatched behind all pieces: a
// piece leaves its partial sums as words of 16 bytes, two values with the two halves of the launch's tag between them, written past the
// caches (agent scope), and a merging workgroup reads the words of its row until all carry the tag.  No counter, fence or flag behind
// the data is needed, a word says itself whether it is there (flags behind the data cost a further way to memory and back: for
// 256 pieces that read 8 MB, us, two launches 4.9, by flags 5.3, by tagged words 4.7).  What bounds it is that way, once there and once
// back.  Words that have come are not asked for again (0.3 us), and the merge is run once over nothing beforehand: its
// instructions come from memory the first time (0.3 us).  Where it is used: merges_itself, with both sides' times.
//
// No result hangs on the order in which workgroups are dispatched or on room for all of them: a merging workgroup looks MERGE_LOOKS times at most
// (0.2 ms).  Then it hands its row over: it writes a flag, a tagged word as well, waits until the flag has arrived, looks once more and, if a piece
// is still missing, leaves.  A piece whose words have arrived looks at the flags of its rows and, where one is set, at all words of the row; if all are there,
// it merges.  Whichever arrives last at memory, a missing piece's last word or the flag, its writer reads the other's afterwards, so one of the two
// merges (both may; they write the same bits).  No piece waits for anything but its own stores, and no other wait is longer than MERGE_LOOKS.
// A piece's way to the flags and back runs beside the merging workgroup's to the piece's words: lists of 1024 and 2048, 32 heads, us, without the flags and with
// them, GPU alone 6.4 and 6.4, 6.9 and 6.9, calls one after the other 6.57 and 6.70, 6.65 and 6.74.
// Before it comes to that, merges_itself keeps the waiting workgroups few: of four launches at a time (the hardware queues of a process), those of three
// leave room on every XCD for the pieces of the fourth.
//
// The tag is 64 random-looking bits that the host draws anew for every call, so whatever the workspace held before is taken for a word of this launch with
// a probability of 2^-64 per word.  A launch captured into a graph would be replayed with the same tag, over words that the replay before left: captured launches
// leave the merge to a second one.  A merging workgroup writes nothing but its own columns of the output.  A lane's aligned 16 bytes are written and read in
// one access.
constexpr int MERGE_COLS = 64;                        // columns of a merging workgroup: two per row (one or four: 0.3, 0.1 us more)
constexpr int MERGE_PARTS = D / MERGE_COLS;
constexpr int MERGE_PIECE_BYTES = (D / 2 + 1) * 16;   // words of a row's piece: its columns, its maximum and sum
constexpr int MERGE_ROW_BYTES = MERGE_PARTS * 16;     // words of a row: its merging workgroups' flags
constexpr int MERGE_LOOKS = 256;
constexpr int MERGE_LDS_FLOATS = 8 * MERGE_COLS + 16 + 1;
constexpr int CACHE_AGENT = 16;                       // cache policy of a buffer access: agent scope (sc1)

__device__ __forceinline__ auto tagged_words(float* base, uint32_t bytes) {
    asm volatile("" : "+s"(base));                       // other workgroups write there too: no longer the __restrict__ argument
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);   // accesses past `bytes` are dropped
}

// One step of the merge: the pieces a thread asked for together join its running (maximum, sum, columns).
template <int U, typename Cols>
__device__ __forceinline__ void fold_pieces(const Cols (&a)[U], const float (&m)[U], const float (&l)[U], const bool (&there)[U], float& mo, float& lo, Cols& ao) {
    float mb = mo;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (there[u]) mb = fmaxf(mb, m[u]);
    if (mb == -INFINITY) return;                     // nothing but empty pieces so far
    const float f0 = (mo == -INFINITY) ? 0.0f : exp2f(mo - mb);
    ao *= f0;
    lo *= f0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        // dropped by select, never by a multiplication: a slot without a piece holds whatever was there before
        const bool live = there[u] && m[u] != -INFINITY;
        const float f = live ? exp2f(m[u] - mb) : 0.0f;
        const Cols au = live ? a[u] : Cols(0.0f);
        ao += au * f;
        lo = __builtin_fmaf(live ? l[u] : 0.0f, f, lo);
    }
    mo = mb;
}

// The eight running merges of a row, one column: their maximum; A and Ls get the column and the sum.
template <typename Col>
__device__ __forceinline__ float meet_in_lds(const float* m, const float* l, Col col, float& A, float& Ls) {
    float M = m[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) M = fmaxf(M, m[j]);
    A = Ls = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float f = (m[j] == -INFINITY) ? 0.0f : exp2f(m[j] - M);
        A = __builtin_fmaf(col(j), f, A);
        Ls = __builtin_fmaf(l[j], f, Ls);
    }
    return M;
}

// A launch's words: rows x n_splits pieces of D / 2 words of columns, as many words of maximum and sum, rows x MERGE_PARTS flags.
struct MergeWords {
    decltype(tagged_words(nullptr, 0)) words;
    uint32_t lo, hi, ml0, flag0;
    int n_splits;

    __device__ __forceinline__ MergeWords(float* base, uint64_t tag, uint32_t rows, int n_splits_)
        : words(tagged_words(base, rows * (n_splits_ * MERGE_PIECE_BYTES + MERGE_ROW_BYTES))), lo((uint32_t)tag), hi((uint32_t)(tag >> 32)),
          ml0(rows * n_splits_ * (D / 2)), flag0(ml0 + rows * n_splits_), n_splits(n_splits_) {}
    __device__ __forceinline__ uint32_t col_at(uint32_t row, uint32_t piece, uint32_t pair) const { return ((row * n_splits + piece) * (D / 2) + pair) * 16u; }
    __device__ __forceinline__ uint32_t ml_at(uint32_t row, uint32_t piece) const { return (ml0 + row * n_splits + piece) * 16u; }
    __device__ __forceinline__ uint32_t flag_at(uint32_t item) const { return (flag0 + item) * 16u; }
    __device__ __forceinline__ u32x4 load(uint32_t at) const { return __builtin_amdgcn_raw_buffer_load_b128(words, at, 0, CACHE_AGENT); }
    __device__ __forceinline__ void store(uint32_t at, float a, float b) const {
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(a), lo, __float_as_uint(b), hi}, words, at, 0, CACHE_AGENT);
    }
    __device__ __forceinline__ bool mine(u32x4 w) const { return w.y == lo && w.w == hi; }
};

// 256 threads look at a row's words, `looks` times at most, and merge its pieces if all are there: the columns of `part`.  Thread (c, sr) has columns
// 2c, 2c + 1 of these and the pieces sr, sr + 8, ...; the eight meet in LDS.  dry: over nothing.  False: words are missing (for the whole workgroup).  ONCE: one look, which
// needs no second set of registers.
template <bool ONCE>
__device__ __forceinline__ bool merge_row(const MergeWords& w, int row, int part, int pieces, int looks, bool dry, uint16_t* __restrict__ out,
                                          float* __restrict__ lse, float* lds) {
    constexpr int WORDS = MERGE_COLS / 2, U = 4;
    const int tid = threadIdx.x, c = tid % WORDS, sr = tid / WORDS;
    float(*const la)[MERGE_COLS] = reinterpret_cast<float(*)[MERGE_COLS]>(lds);
    float* const lm = lds + 8 * MERGE_COLS;
    const int todo = dry ? 1 : pieces;
    float m = -INFINITY, l = 0.0f;
    f32x2 a = {0.0f, 0.0f};
    bool lost = false;
    for (int s0 = sr; s0 - sr < todo; s0 += 8 * U) {
        // What is there (or does not exist) is not asked for again: an address past the buffer's end is no access.
        constexpr uint32_t NOWHERE = 0xfffffff0u;
        u32x4 wa[U], wm[U];
        uint32_t at_a[U], at_m[U];
        bool there[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + 8 * u;
            there[u] = dry || s < pieces;
            at_a[u] = dry || s >= pieces ? NOWHERE : w.col_at(row, s, part * WORDS + c);
            at_m[u] = dry || s >= pieces ? NOWHERE : w.ml_at(row, s);
            wa[u] = wm[u] = u32x4{0u, 0u, 0u, 0u};
        }
        bool ready = false;
        if constexpr (ONCE) {
            bool mine = true;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                wa[u] = w.load(at_a[u]);
                wm[u] = w.load(at_m[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) mine = mine && (at_a[u] == NOWHERE || (w.mine(wa[u]) && w.mine(wm[u])));
            ready = __all(mine);
        }
        for (int look = 0; !ONCE && look < looks && !ready; ++look) {
            asm volatile("" ::: "memory");               // read again
            u32x4 na[U], nm[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                na[u] = w.load(at_a[u]);
                nm[u] = w.load(at_m[u]);
            }
            bool mine = true;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool came = w.mine(na[u]) && w.mine(nm[u]);   // (what was not asked for reads zeros, which no tag is)
                if (came) {
                    wa[u] = na[u];
                    wm[u] = nm[u];
                    at_a[u] = at_m[u] = NOWHERE;
                }
                mine = mine && at_a[u] == NOWHERE;
            }
            ready = __all(mine);
        }
        lost = lost || !ready;
        float mu[U], lu[U];
        f32x2 au[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            au[u] = f32x2{__uint_as_float(wa[u].x), __uint_as_float(wa[u].z)};
            mu[u] = __uint_as_float(wm[u].x);
            lu[u] = __uint_as_float(wm[u].z);
        }
        fold_pieces<U>(au, mu, lu, there, m, l, a);
    }
    *reinterpret_cast<f32x2*>(&la[sr][2 * c]) = a;
    if (c == 0) {
        lm[sr] = lost ? NAN : m;                         // (no piece's maximum is NaN)
        lm[8 + sr] = l;
    }
    lds_barrier();
    bool missing = false;
#pragma unroll
    for (int j = 0; j < 8; ++j) missing = missing || lm[j] != lm[j];
    if (tid < MERGE_COLS) {
        float A, Ls;
        const float M = meet_in_lds(lm, lm + 8, [&](int j) { return la[j][tid]; }, A, Ls);
        const uint16_t res = f32_to_bf16_rne(Ls > 0.0f ? A / Ls : 0.0f);
        if (!dry && !missing) {
            out[(int64_t)row * D + part * MERGE_COLS + tid] = res;
            if (lse && part == 0 && tid == 0) lse[row] = M + log2f(Ls);
        } else {
            asm volatile("" ::"v"((uint32_t)res));
        }
    }
    lds_barrier();                                       // read, before the next round writes
    return !__builtin_amdgcn_readfirstlane(missing);
}

// A merging workgroup: once over nothing, while the pieces are being made, so that the instructions are in the cache when the words are there; then up to
// `looks` looks; then, the row handed over, one more.
__device__ __forceinline__ void wait_and_merge(const MergeWords& w, int item, int pieces, int looks, uint16_t* __restrict__ out, float* __restrict__ lse,
                                               float* lds) {
#pragma nounroll
    for (int round = 0; round < 3; ++round) {
        asm volatile("" : "+s"(round), "+s"(item));      // (each round makes its addresses anew: kept, they cost a wave per SIMD)
        const bool done = merge_row<false>(w, item / MERGE_PARTS, item % MERGE_PARTS, pieces, round == 1 ? looks : 1, round == 0, out, lse, lds);
        if (round == 0) continue;
        if (done) return;
        if (round == 1) {
            float none = 0.0f;
            asm volatile("" : "+v"(none));
            if (threadIdx.x == 0) w.store(w.flag_at(item), none, none);
            asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");   // arrived, before anyone looks again
        }
    }
}

// A piece, behind the stores of its words: the rows row0 .. row0 + n_rows - 1 that were handed over meanwhile, for which this may have been the last piece.
__device__ __forceinline__ void merge_if_handed_over(const MergeWords& w, int row0, int n_rows, int pieces, uint16_t* __restrict__ out,
                                                     float* __restrict__ lse, float* lds) {
    uint32_t* const asked = reinterpret_cast<uint32_t*>(lds + MERGE_LDS_FLOATS - 1);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");   // all of the workgroup's words have arrived
    if (threadIdx.x < 64) {
        const int n_items = n_rows * MERGE_PARTS, lane = threadIdx.x;
        const u32x4 flag = w.load(lane < n_items ? w.flag_at(row0 * MERGE_PARTS + lane) : 0xfffffff0u);
        const uint64_t set = __ballot(lane < n_items && w.mine(flag));
        if (lane == 0) *asked = (uint32_t)set;           // (at most 16 items)
    }
    lds_barrier();
    uint32_t todo = __builtin_amdgcn_readfirstlane(*asked);
    while (__builtin_expect(todo != 0, 0)) {
        const int item = row0 * MERGE_PARTS + __builtin_ctz(todo);
        todo &= todo - 1;
        merge_row<true>(w, item / MERGE_PARTS, item % MERGE_PARTS, pieces, 1, false, out, lse, lds);
    }
}

// SCORE (selection layer, all tokens): the scores of the candidate range [0, L - window) are also
// written to P[b][head][t] (row stride ldp), so the layer's K is read once for both (Alg. 1 computes
// the layer's output and P from the same K).  q.k then runs as the k = 1 MFMA chain -- the pinned
// left-to-right binary32 sum (see "scoring" above) -- instead of the k = 4 bf16 MFMA, and the softmax
// uses those same values.
//
// lse (optional): log2 of each head's softmax denominator, M + log2(l) with scores scaled by
// sm_scale * log2(e); written by whoever writes the head's output (this kernel or the reduce).
//
// PER_HEAD (sparse, GQ = 1): every query head attends its own token list idx[b][head][0 .. cnt[b])
// -- the head-to-head selection the paper compares with (Sec. 3.2, the generalization figure) --
// so a workgroup serves one query head, blockIdx.y counts query heads (G of them) and head y reads
// KV head y >> hshift.  Nothing is shared inside a GQA group: each head fetches its own rows.
template <int GQ, int TI, bool SPARSE, bool PAGED, bool SCORE = false, bool PER_HEAD = false, bool FILTER = false>
__global__ __launch_bounds__(ATTN_THREADS, 2) void attn_kernel(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt, const int32_t* __restrict__ seq_lens,
    const uint16_t* __restrict__ q, int budget, int n_splits, int chunk, int G, uint32_t inv_splits, int n_seqs, float scale_log2e,
    float* __restrict__ part_acc, float* __restrict__ part_ml, uint16_t* __restrict__ out, float* __restrict__ lse,
    uint64_t tag, int looks, int window, int hshift, FilterState flt, KvView kv) {
    static_assert(!(SCORE && SPARSE), "scores are emitted by the pass over all tokens");
    static_assert(!FILTER || SCORE, "the filter is a form of the scoring variant");
    static_assert(!PER_HEAD || (SPARSE && GQ == 1), "per-head token lists: one query head per workgroup");
    constexpr int TILE = TI * 4;                      // tokens per wave iteration (<= 64)
    constexpr int WG_TILE = TILE * ATTN_WAVES;
    constexpr int SETS = (GQ + 3) / 4;                // groups of 4 heads, one MFMA accumulator each
    constexpr int QSB = 136;                          // padded head stride of q in LDS (bf16 elements)
    // A wave's K tile buffer (TILE rows of 256 bytes) also carries its partial accumulators
    // (GQ x 128 floats) into the final merge.
    // The scoring variant parks a tile's K rows in two halves of 64 columns, one after the other (its
    // product chain walks the columns in order anyway), which leaves LDS for the scores of the
    // workgroup's whole run (pstage below).
    constexpr int KSLOTS = SCORE ? 8 : 16;            // 16-byte slots of a K row held in LDS at a time
    constexpr int WAVE_LDS = TILE * KSLOTS * 16;      // bytes of a wave's tile buffer
    static_assert(WAVE_LDS >= GQ * D * 4, "the K tile buffer must hold a wave's partial accumulators");
    __shared__ __attribute__((aligned(16))) unsigned char smem_raw[ATTN_WAVES * WAVE_LDS];
    // this wave's K rows: chunk c of row r at slot c ^ (r & 15) (no bank conflicts in either direction); scoring
    // variant: chunk c (of the half) at slot c ^ ((r >> 1) & 7)
    u32x4* const ktile = reinterpret_cast<u32x4*>(smem_raw) + wave_base_of(threadIdx.x) * (TILE * KSLOTS);
    __shared__ float sm_m[ATTN_WAVES][GQ];
    __shared__ float sm_l[ATTN_WAVES][GQ];
    // A wave's softmax numerators take the place of its K rows once those are scored.  They are
    // stored as bf16 in the operand order of the P.V products below: [row group r][four row loads ig]
    // [set][head][member k], so that the weights of one head for the four tokens a lane multiplies
    // together (rows 4ig .. 4ig+3 of its row group) are one 8-byte word.
    static_assert(TI % 4 == 0 && WAVE_LDS >= TI * SETS * 32, "the numerators must fit the K tile buffer");
    __bf16* const pbuf16 = reinterpret_cast<__bf16*>(ktile);
    // q in LDS: a private bf16 copy per wave, or -- in the scoring variant, whose product chain takes
    // binary32 operands -- one binary32 copy for the workgroup (every wave writes all of it with the
    // same values, so a wave depends on its own writes only and no workgroup barrier is needed).
    constexpr int QSF = 132;                          // padded head stride of the binary32 copy (floats)
    __shared__ __attribute__((aligned(16))) uint16_t qlds_all[SCORE ? 1 : ATTN_WAVES][SCORE ? 8 : SETS * 4 * QSB];
    __shared__ __attribute__((aligned(16))) float qf32[SCORE ? SETS * 4 * QSF : 4];
    // scoring variant: the scores of the workgroup's run (of its last STAGE_IT iterations, should a run be
    // longer: the host caps it at STAGE_TOK tokens), [head][token], on their way to P
    constexpr int STAGE_TOK = GQ >= 8 ? ATTN_SCORE_CHUNK_CAP_G8 : ATTN_SCORE_CHUNK_CAP;   // 32 KB at groups of 4 and 8
    constexpr int STAGE_IT = STAGE_TOK / WG_TILE;
    __shared__ __attribute__((aligned(16))) float pstage[SCORE ? GQ * STAGE_TOK : 4];
    // Filtered form of the scoring variant (FILTER; see sample_threshold_kernel): instead of every score,
    // the buffer takes the (score key, position) composites of the candidates at or above the head's
    // threshold, compacted per head -- STAGE_CAND of them per head at most, or the head is flagged.
    constexpr int STAGE_CAND = STAGE_TOK / 2;         // composites are twice a score's size
    uint64_t* const cstage = reinterpret_cast<uint64_t*>(pstage);
    __shared__ int cand_n[SCORE ? GQ : 1], cand_base[SCORE ? GQ : 1];
    __shared__ uint32_t thr_lds[SCORE ? GQ : 1];
    constexpr bool filtered = FILTER;
    // Workgroups go to the 8 XCDs round-robin in launch order (blockIdx.x fastest).  With ragged
    // lengths the low splits are the busy ones; starting each (sequence, KV head) at a different
    // block spreads them evenly over the XCDs instead of loading the first ones.
    const int gy = blockIdx.y, b = blockIdx.z, H = G * GQ;
    static_assert(sizeof(smem_raw) >= MERGE_LDS_FLOATS * 4, "the merge's sums must fit the tile buffers");
    constexpr bool MERGES = !SCORE && !PER_HEAD && TI == 4;   // forms whose launch may merge its pieces itself: merges_itself asks for short runs
    if constexpr (MERGES) {
        if (__builtin_expect(b >= n_seqs, 0)) {          // behind all pieces: the workgroups that merge them
            const int item = ((b - n_seqs) * G + gy) * (int)gridDim.x + (int)blockIdx.x;
            if (item >= n_seqs * H * MERGE_PARTS) return;
            const int of = item / (H * MERGE_PARTS), pieces = merged_pieces(SPARSE ? min(cnt[of], budget) : seq_lens[of], chunk, n_splits);
            if (pieces > 1)                              // otherwise the only piece writes the result itself
                wait_and_merge(MergeWords(part_acc, tag, n_seqs * H, n_splits), item, pieces, looks, out, lse, reinterpret_cast<float*>(smem_raw));
            return;
        }
    }
    const int kvh = PER_HEAD ? gy >> hshift : gy;
    // (blockIdx.x + pair) % n_splits: inv_splits = (2^32 - 1) / n_splits rounded down, so the quotient is right or one short
    const uint32_t pair = (uint32_t)gy + (uint32_t)G * (uint32_t)b;
    uint32_t turned = blockIdx.x + (pair - __umulhi(pair, inv_splits) * (uint32_t)n_splits);
    if (turned >= (uint32_t)n_splits) turned -= n_splits;
    if (turned >= (uint32_t)n_splits) turned -= n_splits;
    const int split = (int)turned;
    const int tid = threadIdx.x, wave = SCORE ? tid >> 6 : __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r = lane >> 4, c = lane & 15;
    const int begin = split * chunk;
    const int32_t* __restrict__ my_idx = idx + (PER_HEAD ? (int64_t)b * G + gy : (int64_t)b) * budget;
    const int64_t head0 = (int64_t)b * H + gy * GQ;      // first query head of this group
    // Address pipeline.  A row's address is the end of a chain of dependent memory reads: the token
    // list (sparse), then the block table (paged), then the row.  The list entries (posA) of a tile
    // are requested one tile ahead, and so are the pool pages (pgA) of a pass over all tokens, whose
    // positions are arithmetic.  The first entries are fetched here, before the token count is
    // known: a row of idx has `budget` entries, so a read clamped to budget - 1 stays inside it, and
    // entries past the count are masked below like every row past the run's end.
    const int tile0 = begin + wave * TILE;
    int posA[TI], pgA[TI];
    auto idx_load = [&](int t_, int last, int* p) {
        if (SPARSE) {
#pragma unroll
            for (int i = 0; i < TI; ++i) p[i] = my_idx[min(t_ + i * 4 + r, last)];
        }
    };
    idx_load(tile0, budget - 1, posA);

    // Every wave keeps its own bf16 copy of q in LDS (no workgroup barrier on the way in): lane l
    // fetches 16 bytes of head l / 16 per set now and parks them once the first tile's loads are
    // under way.  Heads beyond GQ score zero.
    uint16_t* const qlds = qlds_all[SCORE ? 0 : wave];
    u32x4 qv[SETS];
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        const int h = s * 4 + r;
        qv[s] = *reinterpret_cast<const u32x4*>(q + (head0 + (h < GQ ? h : 0)) * D + c * 8);
        if (h >= GQ) qv[s] = u32x4{0u, 0u, 0u, 0u};
    }
    bool q_parked = false;
    f32x4 acc[SETS][8];                               // [set][column e of the lane's 8]: the four heads of the set
#pragma unroll
    for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            acc[s][e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (!SCORE) asm volatile("" : "+v"(acc[s][e]));   // here, while the token list is on its way, not between the rows' requests
        }
    const int L = seq_lens[b];
    const int n = SPARSE ? min(cnt[b], budget) : L;
    // Everything the first tile's addresses depend on is requested above and has to be here
    // before the first branch; otherwise the compiler sinks each load behind the branch that
    // precedes its first use and the kernel starts with a chain of dependent memory round trips.
    asm volatile("" ::"s"(L), "s"(n), "s"(kv.k), "s"(H));
    // ... nor fetch the arguments that are used later when they are (a round trip each; in the scoring variant the registers they
    // would occupy cost more: 979 -> 983 us for 64 sequences)
    if (!SCORE) asm volatile("" ::"s"(kv.v), "s"(kv.st), "s"(part_acc), "s"(part_ml), "s"(out), "s"(lse), "s"(scale_log2e));
    if (SPARSE) {
#pragma unroll
        for (int i = 0; i < TI; ++i) asm volatile("" ::"v"(posA[i]));
    }
    if (!SCORE) {
#pragma unroll
        for (int s = 0; s < SETS; ++s) asm volatile("" ::"v"(qv[s]));
    }
    if (__builtin_expect(begin >= n, 0)) {               // split >= attn_active_splits(n, chunk), or an empty list:
        if (split == 0) {                                // nothing to attend to
            for (int o = tid; o < GQ * D; o += ATTN_THREADS) out[head0 * D + o] = 0;
            if (lse && tid < GQ) lse[head0 + tid] = -INFINITY;
        }
        return;
    }
    const int end = (begin + chunk < n) ? begin + chunk : n;

    // Scores come from V_MFMA_F32_4X4X4_16B_BF16: per lane four bf16 of q (head = lane % 4)
    // and four of K (the lane's token).  A tile of fewer than 64 tokens has 64 / TILE = PARTS lanes to a token: lane t
    // multiplies part t / TILE of the columns of token t % TILE (32 / PARTS instructions), and two folds over the
    // lane's upper bits add the parts up and leave every lane the whole scores of NZ = 4 SETS / PARTS heads, head0_z
    // onwards -- one (token, head) per lane at 16 tokens and a group of 4, so that the tile's maxima and weights take one
    // chain of operations instead of four and K and q a quarter of the LDS reads.  (When all lanes of a token
    // walked the whole row, reading K and q was what a short run's arithmetic waited for: 4 waves x 16 + 16 reads of 1 KB.  Layer
    // of one sequence, 32 heads, list of 2048: 7.75 -> 7.2 us; 8 sequences, lists of 4096: 27.1 -> 26.6.)
    // The scoring variant's sums run over the columns in order: one part, every lane all heads (lanes beyond TILE repeat a token
    // and add nothing to l).
    constexpr int PARTS = SCORE ? 1 : 64 / TILE;
    constexpr int NV = SETS * 4, NZ = PARTS == 1 ? GQ : NV / PARTS;
    static_assert(PARTS == 1 || PARTS == 2 || PARTS == 4, "tiles of 16, 32 or 64 tokens");
    const int tl = lane % TILE;
    const bool owner = PARTS > 1 || lane < TILE;
    const int head0_z = PARTS == 1 ? 0 : PARTS == 2 ? (lane >> 5) * (NV / 2) : (lane >> 5) * (NV / 2) + ((lane >> 4) & 1) * (NV / 4);
    // token tl is row load (tl / 4) of row group (tl % 4): where its numerators go (bf16 elements)
    const int p_slot = (((tl & 3) * (TI / 4) + (tl >> 4)) * SETS * 4 + head0_z) * 4 + ((tl >> 2) & 3);
    float m[NZ], l[NZ];                               // of the lane's heads
#pragma unroll
    for (int v = 0; v < NZ; ++v) {
        m[v] = LOWEST;
        l[v] = 0.0f;
    }

    // Rows past the end of the run read some token of the sequence (a valid row) so that all
    // loads are unconditional and issue back to back; their scores are masked below.
    // The next tile's K rows are requested as soon as this tile's are parked in LDS, i.e. before
    // this tile's arithmetic (not in the scoring variant, whose
    // 64-token tiles leave no registers for it; there the rows are requested at the top of the tile's own iteration).
    // The K rows are requested whether there is a next tile or not (rows past the run's end are the run's last): loads return
    // in order, a wait counts those that may still be under way, and behind a branch the compiler cannot count them -- it
    // waited for the next tile's K rows before it multiplied this tile's V rows.  (With that, the accumulators cleared while the
    // token list is on its way and the tail's arguments fetched at the start: list of 2048 7.2 -> 6.95 us, 64 heads and 4096 9.6 ->
    // 8.4; all of 32768 tokens, 32 heads, 26.2 -> 25.3; 8 sequences of 16384 86.8 -> 84.9.)
    constexpr bool PREFETCH = !SCORE;
    // The scoring variant of a group of 8 has no registers for K and V rows at once (64 each at 64-token
    // tiles, beside 64 accumulators): its V rows are requested once the K rows are parked in LDS.
    constexpr bool V_LATE = SCORE && (GQ >= 8 || (FILTER && GQ >= 4));
    u32x4 kreg[TI], vreg[TI];
    int64_t off[TI];
    // a valid position for row load i of the tile that starts at list entry t_ (an index outside the
    // sequence is a caller error; never fault on it)
    auto tile_pos = [&](int t_, int i, const int* p) {
        return (uint32_t)(SPARSE ? max(min(p[i], L - 1), 0) : min(t_ + i * 4 + r, end - 1));
    };
    // Pool pages of the tile's rows.  A pass over all tokens walks the table in order: tiles start at
    // multiples of 16 tokens, so row loads 4ig .. 4ig+3 of every lane fall into one page, entry
    // (t_ / 16 + ig) of the table (rows clamped to the run's last token: that token's page), and only
    // TI / 4 wave-uniform entries are fetched (g[ig]).
    auto page_load = [&](int t_, const int* p, int* g) {
        if constexpr (PAGED && SPARSE) {
#pragma unroll
            for (int i = 0; i < TI; ++i) g[i] = kv.bt[(int64_t)b * kv.max_pages + (tile_pos(t_, i, p) >> 4)];
        } else if constexpr (PAGED) {
#pragma unroll
            for (int ig = 0; ig < TI / 4; ++ig)
                g[ig] = kv.bt[(int64_t)b * kv.max_pages + min((t_ >> 4) + ig, (end - 1) >> 4)];
        }
    };
    auto make_off = [&](int t_, const int* p, int* g) {
        if constexpr (SPARSE && PAGED) page_load(t_, p, g);
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            const uint32_t pos = tile_pos(t_, i, p);
            if (PAGED) off[i] = (((int64_t)g[SPARSE ? i : i >> 2] * kv.G + kvh) * PAGE + (pos & (PAGE - 1))) * D + c * 8;
            else off[i] = (int64_t)b * kv.sb + (int64_t)kvh * kv.sh + (int64_t)pos * kv.st + c * 8;
        }
    };
    auto request_k = [&]() {
#pragma unroll
        for (int i = 0; i < TI; ++i) kreg[i] = row_load<PER_HEAD>(kv.k + off[i]);
    };
    auto request_v = [&]() {
#pragma unroll
        for (int i = 0; i < TI; ++i) vreg[i] = row_load<PER_HEAD>(kv.v + off[i]);
    };
    // After the rows of the tile at t_ have been requested: the lookups for the tile after it.
    auto advance = [&](int t_) {
        idx_load(t_ + WG_TILE, end - 1, posA);           // (past the run's end: its last row, not rows of the next run)
        if constexpr (!SPARSE) page_load(t_ + WG_TILE, posA, pgA);   // sparse: looked up where the offsets are made
    };
    if constexpr (!SPARSE) page_load(tile0, posA, pgA);
    auto park_q = [&]() {
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            if constexpr (SCORE) {
                float qf[8];
                unpack8(make_uint4(qv[s].x, qv[s].y, qv[s].z, qv[s].w), qf);
                float* const dst = &qf32[(s * 4 + r) * QSF + c * 8];
                *reinterpret_cast<f32x4*>(dst) = f32x4{qf[0], qf[1], qf[2], qf[3]};
                *reinterpret_cast<f32x4*>(dst + 4) = f32x4{qf[4], qf[5], qf[6], qf[7]};
            } else {
                *reinterpret_cast<u32x4*>(&qlds[(s * 4 + r) * QSB + c * 8]) = qv[s];
            }
        }
    };
    if constexpr (PREFETCH) {
        make_off(tile0, posA, pgA);
        request_k();
        advance(tile0);
        __builtin_amdgcn_sched_barrier(0);
        park_q();
    }
    // Scoring variant: the scores go to P through a staging buffer in LDS that the whole workgroup
    // writes out in one burst.  A few per cent of small writes scattered
    // through a streaming read cost this machine a sixth of its read rate; the same bytes written in
    // workgroup-sized bursts cost a third of that (measured with plain read / write kernels).  The
    // burst is issued at the end of the workgroup's run (the host caps a run at STAGE_TOK tokens; a
    // longer one would take a burst every STAGE_IT iterations, before the next tile's rows are
    // requested).  Measured on the selection pass, us without stores / scattered stores / bursts:
    // c3 95 / 106 / 99, c4 100 / 121 / 106, c5 867 / 1036 / 1008.  Giving every workgroup its own
    // burst phase, so that the chip's bursts do not coincide, was measured too and is slower.
    auto flush_scores = [&](int g0, int n_tok) {       // staged tokens [g0, g0 + n_tok) of this workgroup's run
        if constexpr (SCORE) {
            const int lim = min(end, L - window);      // candidates only; L <= budget: rho is every token, nothing is scored
            if (L > budget && g0 < lim) {
                const int quads = n_tok >> 2;
                for (int i = tid; i < GQ * quads; i += ATTN_THREADS) {
                    const int h = i / quads, w4 = (i - h * quads) * 4, t = g0 + w4;
                    const f32x4 v = *reinterpret_cast<const f32x4*>(&pstage[h * STAGE_TOK + w4]);
                    float* const dst = &flt.scores[(head0 + h) * flt.cap + t];
                    if (t + 3 < lim) {
                        __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(dst));
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (t + e < lim) dst[e] = v[e];
                    }
                }
            }
        }
    };
    // filtered form: the staged candidates of every head go to the head's list in memory, one reservation
    // per head and workgroup.  The reservation is a device-scope atomic whose answer takes microseconds:
    // reserve_candidates asks (thread h for head h; returns the answer, -1 if there is nothing to copy),
    // copy_candidates uses the answer and empties the buffer -- at the end of a run the workgroup merges
    // and writes its attention partials in between.  Both are called by the whole workgroup.
    auto reserve_candidates = [&]() -> int {
        int base = -1;
        if constexpr (SCORE) {
            lds_barrier();                               // every wave's candidates are staged
            if (tid < GQ) {
                const int n_h = cand_n[tid];
                if (n_h > STAGE_CAND) flag_failed(flt, head0 + tid);   // more candidates than the buffer held: some are lost
                else if (n_h > 0) base = atomicAdd(&flt.cand_cnt[head0 + tid], n_h);
            }
        }
        return base;
    };
    auto copy_candidates = [&](int base) {
        if constexpr (SCORE) {
            if (tid < GQ) {
                if (base >= 0 && base + cand_n[tid] > flt.cap) {   // the head's list is full (the count stays above cap: the ranking sees it too)
                    flag_failed(flt, head0 + tid);
                    base = -1;
                }
                cand_base[tid] = base;
            }
            lds_barrier();
#pragma unroll
            for (int h = 0; h < GQ; ++h) {
                const int n_h = cand_n[h], base_h = cand_base[h];
                if (base_h >= 0) {
                    uint64_t* const dst = flt.cand + (head0 + h) * flt.cap + base_h;
                    for (int i = tid; i < n_h; i += ATTN_THREADS) __builtin_nontemporal_store(cstage[h * STAGE_CAND + i], &dst[i]);
                }
            }
            lds_barrier();                               // all read, before the counters start again
            if (tid < GQ) cand_n[tid] = 0;
            lds_barrier();
        }
    };
    if constexpr (FILTER) {                              // the heads' thresholds wait in LDS, not in registers
        if (tid < GQ) {
            thr_lds[tid] = flt.thr[head0 + tid];
            cand_n[tid] = 0;
        }
        lds_barrier();
    }
    int t_opaque = 0;                                    // always zero, unknown to the compiler
    int it_staged = 0;                                   // first iteration whose scores are still in the staging buffer
    int it = 0;                                          // iterations of the workgroup so far
    // (Without the scoring variant's barriers every wave leaves when its own tiles are done.)
    for (int w0 = SCORE ? begin : tile0; w0 < end; w0 += WG_TILE, ++it) {
        const int t0 = SCORE ? w0 + wave * TILE : w0;
        // Only the scoring variant has workgroup barriers inside the loop; there a wave whose tile lies
        // past the run's end still takes part in them.
        const bool active = t0 < end;
        // workgroup-uniform; the buffer holds STAGE_IT iterations at most
        const bool burst_due = SCORE && it - it_staged == STAGE_IT;
        if (burst_due) {
            if (filtered) {
                copy_candidates(reserve_candidates());
            } else {
                lds_barrier();                           // every wave's scores since the last burst are staged
                flush_scores(begin + it_staged * WG_TILE, (it - it_staged) * WG_TILE);
                lds_barrier();                           // ... and read, before the buffer is written again
            }
            it_staged = it;
        }
        if (SCORE && !active) continue;
        if constexpr (!PREFETCH) {
            make_off(t0, posA, pgA);
            // K rows first: they are needed first (parked in LDS and scored), and loads return in
            // order, so the scores are under way while the V rows are still arriving.
            request_k();
        }
        if constexpr (!V_LATE) request_v();
        if constexpr (!PREFETCH && !V_LATE) advance(t0);
        __builtin_amdgcn_sched_barrier(0);               // keep every load above the arithmetic
        if (SCORE && !q_parked) {
            park_q();
            q_parked = true;
        }
        if constexpr (!SCORE) {
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int row = i * 4 + r;
                ktile[row * 16 + (c ^ (row & 15))] = kreg[i];
            }
            wave_lds_sync();
        }
        if constexpr (PREFETCH) {
            make_off(t0 + WG_TILE, posA, pgA);
            request_k();
            advance(t0 + WG_TILE);
            __builtin_amdgcn_sched_barrier(0);
        }

        f32x4 sc[SETS];
#pragma unroll
        for (int s = 0; s < SETS; ++s) sc[s] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (SCORE) {
            // columns 0..63, then 64..127: the lanes holding that half of a row park it, every lane then
            // walks its own token's 64 columns in order
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (half) wave_lds_sync();            // the first half has been read
                if ((c >> 3) == half) {
#pragma unroll
                    for (int i = 0; i < TI; ++i) {
                        const int row = i * 4 + r;
                        ktile[row * 8 + ((c & 7) ^ ((row >> 1) & 7))] = kreg[i];
                    }
                }
                wave_lds_sync();
                if constexpr (V_LATE) {
                    if (half) {                       // the K rows' registers are free now
                        // the offsets are made again rather than kept in 32 registers since the K requests;
                        // the compiler must not see that they are the same values, or it keeps them
                        asm volatile("" : "+v"(t_opaque));
                        make_off(t0 + t_opaque, posA, pgA);
                        request_v();
                        advance(t0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
#pragma unroll
                for (int c8 = 0; c8 < 8; ++c8) {
                    const int cc = half * 8 + c8;
                    const u32x4 kw = ktile[tl * 8 + (c8 ^ ((tl >> 1) & 7))];
                    float kf[8];
                    unpack8(make_uint4(kw.x, kw.y, kw.z, kw.w), kf);
                    float qf[SETS][8];
#pragma unroll
                    for (int s = 0; s < SETS; ++s) {
                        const float* const src = &qf32[(s * 4 + (lane & 3)) * QSF + cc * 8];
                        const f32x4 qa = *reinterpret_cast<const f32x4*>(src), qb = *reinterpret_cast<const f32x4*>(src + 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            qf[s][e] = qa[e];
                            qf[s][4 + e] = qb[e];
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e)
#pragma unroll
                        for (int s = 0; s < SETS; ++s)
                            sc[s] = __builtin_amdgcn_mfma_f32_4x4x1f32(qf[s][e], kf[e], sc[s], 0, 0, 0);
                }
            }
            if (filtered) {
                const int t = t0 + tl;
                const bool is_cand = lane < TILE && t >= flt.n_sink && t < min(end, L - window);
#pragma unroll
                for (int h = 0; h < GQ; ++h) {
                    const uint32_t key = score_key(sc[h >> 2][h & 3]), thr = thr_lds[h];
                    const bool keep = is_cand && thr != 0xffffffffu && key >= thr;
                    const uint64_t kept = __ballot(keep);
                    if (kept) {                          // wave-uniform: one reservation per wave and head
                        int base = 0;
                        if (lane == 0) base = atomicAdd(&cand_n[h], __popcll(kept));
                        base = __builtin_amdgcn_readfirstlane(base);
                        const int slot = base + mbcnt(kept);
                        if (keep && slot < STAGE_CAND) cstage[h * STAGE_CAND + slot] = ((uint64_t)key << 32) | (uint32_t)~(uint32_t)t;
                    }
                    asm volatile("" ::: "memory");       // one head at a time: nothing of the next is fetched early
                }
            } else if (lane < TILE) {
#pragma unroll
                for (int h = 0; h < GQ; ++h) pstage[h * STAGE_TOK + (it - it_staged) * WG_TILE + wave * TILE + tl] = sc[h >> 2][h & 3];
            }
        } else {
            // This lane's part of the columns, in quarters of a row; the two halves of a chunk into sums of their own (shorter chains).  A score is
            // (q0 + q1) + (q2 + q3) of its quarters whatever the tile's width -- two of them in a lane (tiles of 32 tokens), or one, the folds' first
            // step pairing lanes 32 apart --, so that a token weighs the same in passes over many tokens and over few: the recall of a set
            // is a ratio of two such passes (at scores of 2^20 it came out as infinity with sums of the lanes' own order).
            constexpr int QUARTERS = 4 / PARTS;
            const int of = lane / TILE, part0 = (PARTS == 4 ? (of & 1) * 2 + (of >> 1) : of * 2) * 4, slot0 = part0 ^ (tl & 15);
#pragma unroll
            for (int qd = 0; qd < QUARTERS; ++qd) {
                f32x4 lo[SETS], hi[SETS];
#pragma unroll
                for (int s = 0; s < SETS; ++s) lo[s] = hi[s] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int j = qd * 4; j < qd * 4 + 4; ++j) {
                    const u32x4 kw = ktile[tl * 16 + (slot0 ^ j)];
                    const s16x4 klo = __builtin_bit_cast(s16x4, make_uint2(kw.x, kw.y)), khi = __builtin_bit_cast(s16x4, make_uint2(kw.z, kw.w));
#pragma unroll
                    for (int s = 0; s < SETS; ++s) {
                        const u32x4 qw = *reinterpret_cast<const u32x4*>(&qlds[(s * 4 + (lane & 3)) * QSB + (part0 + j) * 8]);
                        lo[s] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, make_uint2(qw.x, qw.y)), klo, lo[s], 0, 0, 0);
                        hi[s] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, make_uint2(qw.z, qw.w)), khi, hi[s], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int s = 0; s < SETS; ++s) sc[s] = qd == 0 ? lo[s] + hi[s] : sc[s] + (lo[s] + hi[s]);
            }
        }
        float z[NZ];                                  // the lane's scores: token tl, heads head0_z ...
        if constexpr (PARTS == 1) {
#pragma unroll
            for (int v = 0; v < NZ; ++v) z[v] = sc[v >> 2][v & 3];
        } else {
            float y[NV / 2];
#pragma unroll
            for (int v = 0; v < NV / 2; ++v) y[v] = fold_halves(sc[v >> 2][v & 3], sc[(v + NV / 2) >> 2][(v + NV / 2) & 3]);
#pragma unroll
            for (int v = 0; v < NZ; ++v) {
                if constexpr (PARTS == 2) z[v] = y[v];
                else z[v] = fold_rows(y[v], y[v + NV / 4]);
            }
        }
        const bool valid = t0 + tl < end;
        float corr[NZ];
#pragma unroll
        for (int v = 0; v < NZ; ++v) {
            const float zs = valid ? z[v] * scale_log2e : -INFINITY;
            float mt = row_max16(zs);                 // over the lanes that hold the same heads
            if (TILE > 16) mt = max_with_row_neighbour(mt);
            if (TILE > 32 || PARTS == 1) mt = max_with_other_half(mt);
            const float m_new = fmaxf(m[v], mt);
            // (exp2f, not the instruction alone, here and in the merges: the instruction makes zero of weights below 2^-126, which beside a
            // value of 2^120 are not nothing.  16 sequences of 8192, us, the instruction and exp2f: 32 heads 82.7 and 83.2, 64 84.0 and 84.6; a step
            // of 32 layers, lists of 2048: 364 and 373)
            corr[v] = exp2f(m[v] - m_new);
            m[v] = m_new;
            // the weight enters numerator and denominator as the same bf16 value
            const __bf16 pb = (__bf16)exp2f(zs - m_new);
            pbuf16[p_slot + v * 4] = pb;
            l[v] = l[v] * corr[v] + (owner ? (float)pb : 0.0f);
        }
#pragma unroll
        for (int h = 0; h < GQ; ++h) {
            const float ch = PARTS == 1 ? corr[h] : lane_value(corr[h % NZ], h / NZ * (64 / PARTS));
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[h >> 2][e][h & 3] *= ch;
        }
        wave_lds_sync();
        __builtin_amdgcn_sched_barrier(0);               // nothing waits for V rows before the weights are made
        // P.V on the matrix cores, four tokens per instruction.  A lane holds columns 8c .. 8c+7 of the
        // rows i*4 + r; the same column of four of its rows (4ig .. 4ig+3) is gathered into one bf16
        // quadruple (V_PERM_B32), which is this lane's column of the 4 x 4 B operand; the A operand is
        // the four tokens' weights of head (lane % 4).  One V_MFMA_F32_4X4X4_16B_BF16 then adds, for the
        // lane's column, the four tokens' products of four heads to the binary32 accumulator.
#pragma unroll
        for (int ig = 0; ig < TI / 4; ++ig) {
            s16x4 pa[SETS];
#pragma unroll
            for (int s = 0; s < SETS; ++s)
                pa[s] = *reinterpret_cast<const s16x4*>(pbuf16 + (((r * (TI / 4) + ig) * SETS + s) * 4 + (lane & 3)) * 4);
#pragma unroll
            for (int w2 = 0; w2 < 4; ++w2) {
                const uint32_t r0 = vreg[4 * ig][w2], r1 = vreg[4 * ig + 1][w2], r2 = vreg[4 * ig + 2][w2], r3 = vreg[4 * ig + 3][w2];
                const uint2 lo = make_uint2(__builtin_amdgcn_perm(r1, r0, 0x05040100u), __builtin_amdgcn_perm(r3, r2, 0x05040100u));
                const uint2 hi = make_uint2(__builtin_amdgcn_perm(r1, r0, 0x07060302u), __builtin_amdgcn_perm(r3, r2, 0x07060302u));
                const s16x4 vlo = __builtin_bit_cast(s16x4, lo), vhi = __builtin_bit_cast(s16x4, hi);
#pragma unroll
                for (int s = 0; s < SETS; ++s) {
                    acc[s][2 * w2] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(pa[s], vlo, acc[s][2 * w2], 0, 0, 0);
                    acc[s][2 * w2 + 1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(pa[s], vhi, acc[s][2 * w2 + 1], 0, 0, 0);
                }
            }
        }
        wave_lds_sync();                              // the tile buffers are rewritten next iteration
    }
    int cand_reserved = -1;
    if constexpr (SCORE) {
        if (filtered) {
            cand_reserved = reserve_candidates();        // used after the merge below
        } else if (it > it_staged) {                   // the iterations staged since the last burst
            lds_barrier();
            flush_scores(begin + it_staged * WG_TILE, (it - it_staged) * WG_TILE);
        }
    }
    // Merge.  Inside the wave the four row groups are folded with lane swaps: of the N = 8 GQ
    // values of a lane, two folds leave N / 4 complete sums, those with flat index (head * 8 +
    // column) v0 .. v0 + N/4 - 1 where v0 depends on the row group.  The wave parks them in its
    // own tile buffer and the four waves meet in LDS.
    constexpr int N = GQ * 8;
    float* const wsum = reinterpret_cast<float*>(ktile);           // [GQ][D] of this wave
    {
        float y[N / 2], z[N / 4];
#pragma unroll
        for (int v = 0; v < N / 2; ++v) {
            constexpr int HALF = N / 2;                  // flat index = head * 8 + column
            y[v] = fold_halves(acc[v >> 5][v & 7][(v >> 3) & 3], acc[(v + HALF) >> 5][(v + HALF) & 7][((v + HALF) >> 3) & 3]);
        }
#pragma unroll
        for (int v = 0; v < N / 4; ++v) z[v] = fold_rows(y[v], y[v + N / 4]);
        const int v0 = (r >> 1) * (N / 2) + (r & 1) * (N / 4);
        if (N / 4 >= 4) {
#pragma unroll
            for (int j = 0; j < N / 16; ++j) {
                const int v = v0 + 4 * j;
                *reinterpret_cast<f32x4*>(&wsum[(v >> 3) * D + c * 8 + (v & 7)]) = f32x4{z[4 * j], z[4 * j + 1], z[4 * j + 2], z[4 * j + 3]};
            }
        } else {
            *reinterpret_cast<f32x2*>(&wsum[c * 8 + v0]) = f32x2{z[0], z[1]};
        }
    }
#pragma unroll
    for (int v = 0; v < NZ; ++v) {
        float ls = row_sum16(l[v]);
        if (TILE > 16) ls = fold_rows(ls, ls);
        if (PARTS == 1) ls = fold_halves(ls, ls);
        const int h = head0_z + v;
        if (lane % (64 / PARTS) == 0 && (PARTS == 1 || h < GQ)) {
            sm_m[wave][h] = m[v];
            sm_l[wave][h] = ls;
        }
    }
    __syncthreads();
    const float* const sums = reinterpret_cast<const float*>(smem_raw);
    // a thread has PER consecutive columns of a head (threads beyond GQ * D / PER: none)
    constexpr int PER = GQ * D >= 2 * ATTN_THREADS ? GQ * D / ATTN_THREADS : 2;
    typedef float f32_per __attribute__((ext_vector_type(PER)));
    typedef uint16_t u16_per __attribute__((ext_vector_type(PER)));
    if (tid * PER < GQ * D) {
        const int o = tid * PER, h = o / D, col = o % D;
        f32_per part[ATTN_WAVES];
        float mw[ATTN_WAVES], lw[ATTN_WAVES];
#pragma unroll
        for (int wv = 0; wv < ATTN_WAVES; ++wv) {
            mw[wv] = sm_m[wv][h];
            lw[wv] = sm_l[wv][h];
            part[wv] = *reinterpret_cast<const f32_per*>(&sums[wv * (WAVE_LDS / 4) + o]);
        }
        const float M = fmaxf(fmaxf(mw[0], mw[1]), fmaxf(mw[2], mw[3]));
        f32_per A = part[0] * exp2f(mw[0] - M);
        float Ls = lw[0] * exp2f(mw[0] - M);
#pragma unroll
        for (int wv = 1; wv < ATTN_WAVES; ++wv) {
            const float f = exp2f(mw[wv] - M);
#pragma unroll
            for (int e = 0; e < PER; ++e) A[e] = __builtin_fmaf(part[wv][e], f, A[e]);
            Ls = __builtin_fmaf(lw[wv], f, Ls);
        }
        if (n <= chunk) {                                // this workgroup saw the whole token list
            u16_per res;
#pragma unroll
            for (int e = 0; e < PER; ++e) res[e] = f32_to_bf16_rne(Ls > 0.0f ? A[e] / Ls : 0.0f);
            uint16_t* const dst = out + (head0 + h) * D + col;
            if ((uintptr_t)out % sizeof(u16_per) == 0) {
                *reinterpret_cast<u16_per*>(dst) = res;
            } else {
#pragma unroll
                for (int e = 0; e < PER; ++e) dst[e] = res[e];
            }
            if (lse && col == 0) lse[head0 + h] = M + log2f(Ls);
        } else if (MERGES && tag) {         // for a merging workgroup of this launch
            const MergeWords w(part_acc, tag, n_seqs * H, n_splits);
#pragma unroll
            for (int e = 0; e < PER; e += 2) w.store(w.col_at(head0 + h, split, (col + e) / 2), A[e], A[e + 1]);
            if (col == 0) w.store(w.ml_at(head0 + h, split), M, Ls);
        } else {
            const int64_t p = (head0 + h) * n_splits + split;
            *reinterpret_cast<f32_per*>(&part_acc[p * D + col]) = A;
            if (col == 0) *reinterpret_cast<f32x2*>(&part_ml[p * 2]) = f32x2{M, Ls};
        }
    }
    if constexpr (MERGES) {
        if (tag && n > chunk)
            merge_if_handed_over(MergeWords(part_acc, tag, n_seqs * H, n_splits), (int)head0, GQ, merged_pieces(n, chunk, n_splits), out, lse,
                                 reinterpret_cast<float*>(smem_raw));
    }
    if constexpr (FILTER) copy_candidates(cand_reserved);
}

// ---------------------------------------------------------------- scoring pass
//
// P[b][h][t] = q_h . K_t, grid (n_splits, G, B), 256 threads.  A workgroup takes every n_splits-th workgroup tile -- one, as a
// rule -- of a (sequence, KV head), a wave TI * 4 tokens of it.  A K row is read by 16 lanes with one 16-byte load each;
// the wave parks its rows in LDS in two halves of 64 columns (8 KB instead of 16 per 64 tokens: the product chain walks the
// columns in order anyway) and every lane reads its own token's columns back.  The tile's scores take the place of its rows and are
// written by the whole workgroup, 1 KB of a head at a time.
//
// What bounds it is memory, if enough loads are in flight while tiles are worked on.  Nothing is requested ahead inside a
// workgroup: it has one tile and four workgroups share a CU, 256 KB of rows, whose waits and arithmetic overlap.
// Measured against two workgroups with runs of 512 to 2048 tokens, q in registers and the next tile's rows on their way
// (us; 8 pairs of 32768, 64 of 16384, 8 of 131072 with groups of 8): 16.1, 47.2, 63.3 -> 14.5, 46.2, 53.0; with both tiles' rows
// in registers 17.3, 49.6, 61.2.
//
// all: every token of every sequence is scored (a selection layer, whose values weigh them all); otherwise the
// candidate range [0, L - window) of the sequences longer than the budget (cusa_select, the filtered selection's second
// chance: with flt.fail set only the groups that have a flagged head, and nothing when the counter is 0).
// keep: P is small enough for the last-level cache to hold until the top-k reads it (ordinary stores, SCORE_KEEP_BYTES).
template <int GQ, int TI, bool PAGED>
__global__ __launch_bounds__(ATTN_THREADS, 4) void score_kernel(const int32_t* __restrict__ seq_lens, const uint16_t* __restrict__ q,
                                                                 int budget, int window, int n_splits, int G, int all, int keep,
                                                                 float* __restrict__ P, int64_t ldp, FilterState flt, KvView kv) {
    constexpr int TILE = TI * 4, WG_TILE = TILE * ATTN_WAVES;
    constexpr int SETS = (GQ + 3) / 4;
    constexpr int QSF = 132;                          // padded head stride of q in LDS (floats)
    static_assert(GQ * TILE * 4 <= TILE * 128, "a tile's scores take the place of its rows");
    __shared__ __attribute__((aligned(16))) u32x4 ktile_all[ATTN_WAVES][TILE * 8];   // chunk c of a row's half at slot c ^ ((row >> 1) & 7)
    __shared__ __attribute__((aligned(16))) float qf32[SETS * 4 * QSF];   // binary32; every wave writes all of it, no barrier
    if (!all && flt.fail && *flt.n_failed == 0) return;
    const int kvh = blockIdx.y, b = blockIdx.z;
    // workgroups go to the 8 XCDs round-robin: short sequences' idle ones are spread over them
    const int split = (int)((blockIdx.x + kvh + G * b) % (unsigned)n_splits);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t head0 = ((int64_t)b * G + kvh) * GQ;
    const int L = uniform_load(seq_lens + b);
    if (!all) {
        if (L <= budget) return;                      // rho is every token: nothing is scored
        if (flt.fail) {
            int any = 0;
#pragma unroll
            for (int h = 0; h < GQ; ++h) any |= flt.fail[head0 + h];
            if (!any) return;
        }
    }
    const int n = all ? L : L - window;
    const int last = n - 1;
    u32x4* const ktile = ktile_all[wave];
    float* const stage = reinterpret_cast<float*>(ktile);   // [GQ][TILE]
    int my_lane = lane;
    for (int w0 = split * WG_TILE; w0 <= last; w0 += n_splits * WG_TILE) {
        const int t0 = w0 + wave * TILE;
        asm volatile("" : "+v"(my_lane));             // what is made of it is made where it is needed: there are no registers to keep it
        const int r = my_lane >> 4, c = my_lane & 15;
        u32x4 qv[SETS];                               // lane: 16 bytes of head 4s + r; heads beyond the group score zero
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            const int h = s * 4 + r;
            qv[s] = *reinterpret_cast<const u32x4*>(q + (head0 + (h < GQ ? h : 0)) * D + c * 8);
            if (h >= GQ) qv[s] = u32x4{0u, 0u, 0u, 0u};
        }
        // rows past the end are the last token's; their scores are not written
        u32x4 kreg[TI];
#pragma unroll
        for (int ig = 0; ig < TI / 4; ++ig) {         // 16 rows: one page
            if constexpr (PAGED) {
                const int first = min(t0 + 16 * ig, last & ~15), rows = last - first;
                const int64_t page = uniform_load(kv.bt + (int64_t)b * kv.max_pages + (first >> 4));
                const uint16_t* const at = kv.k + (page * kv.G + kvh) * (PAGE * D);
#pragma unroll
                for (int i = 0; i < 4; ++i) kreg[4 * ig + i] = stream_load(at + (uint32_t)(min(i * 4 + r, rows) * D + c * 8));
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int pos = min(t0 + (4 * ig + i) * 4 + r, last);
                    kreg[4 * ig + i] = stream_load(kv.k + ((int64_t)b * kv.sb + (int64_t)kvh * kv.sh + (int64_t)pos * kv.st + c * 8));
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < SETS; ++s) {              // (again for every tile, with the same values: there is one as a rule)
            float qf[8];
            unpack8(make_uint4(qv[s].x, qv[s].y, qv[s].z, qv[s].w), qf);
            float* const dst = &qf32[(s * 4 + r) * QSF + c * 8];
            *reinterpret_cast<f32x4*>(dst) = f32x4{qf[0], qf[1], qf[2], qf[3]};
            *reinterpret_cast<f32x4*>(dst + 4) = f32x4{qf[4], qf[5], qf[6], qf[7]};
        }
        const int tl = my_lane % TILE;                // the token of the tile that this lane scores
        f32x4 sc[SETS];
#pragma unroll
        for (int s = 0; s < SETS; ++s) sc[s] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (half) wave_lds_sync();                // the first half has been read
            if ((c >> 3) == half) {
#pragma unroll
                for (int i = 0; i < TI; ++i) {
                    const int row = i * 4 + r;
                    ktile[row * 8 + ((c & 7) ^ ((row >> 1) & 7))] = kreg[i];
                }
            }
            wave_lds_sync();
#pragma unroll
            for (int c8 = 0; c8 < 8; ++c8) {
                const int cc = half * 8 + c8;
                const u32x4 kw = ktile[tl * 8 + (c8 ^ ((tl >> 1) & 7))];
                float kf[8];
                unpack8(make_uint4(kw.x, kw.y, kw.z, kw.w), kf);
                float qf[SETS][8];
#pragma unroll
                for (int s = 0; s < SETS; ++s) {
                    const float* const src = &qf32[(s * 4 + (my_lane & 3)) * QSF + cc * 8];
                    const f32x4 qa = *reinterpret_cast<const f32x4*>(src), qb = *reinterpret_cast<const f32x4*>(src + 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        qf[s][e] = qa[e];
                        qf[s][4 + e] = qb[e];
                    }
                }
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int s = 0; s < SETS; ++s) sc[s] = __builtin_amdgcn_mfma_f32_4x4x1f32(qf[s][e], kf[e], sc[s], 0, 0, 0);
                if (SETS == 2 || (c8 & 1)) __builtin_amdgcn_sched_barrier(0);   // (no further ahead: registers)
            }
        }
        wave_lds_sync();                              // the rows have been read
        asm volatile("" : "+v"(my_lane));
        if (my_lane < TILE) {
#pragma unroll
            for (int h = 0; h < GQ; ++h) stage[h * TILE + my_lane] = sc[h >> 2][h & 3];
        }
        lds_barrier();
        constexpr int QUADS = WG_TILE / 4;
        for (int i = wave * 64 + my_lane; i < GQ * QUADS; i += ATTN_THREADS) {
            const int h = i / QUADS, w4 = (i % QUADS) * 4, t = w0 + w4;
            const f32x4 v = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(ktile_all[w4 / TILE]) + h * TILE + w4 % TILE);
            float* const dst = &P[(head0 + h) * ldp + t];
            if (t + 3 <= last) {
                if (keep) *reinterpret_cast<f32x4*>(dst) = v;   // uniform
                else __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(dst));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (t + e <= last) dst[e] = v[e];
            }
        }
        if (w0 + n_splits * WG_TILE <= last) lds_barrier();   // read, before the tile buffers are written again
    }
}

// ---------------------------------------------------------------- a selection layer's values
//
// out = softmax(scale * P) V for the scores P that score_kernel left: the second half of a selection layer's full attention.
// It does not enter the selection, so its workgroups share a launch with the top-k's (topk_values_kernel): those keep a CU
// each busy with latencies, these stream V meanwhile.
//
// A workgroup of 16 waves owns a run of tokens of one (sequence, KV head); a wave takes tiles of 16 tokens: 16 lanes per 256-byte
// row, four row loads.  Lane (row group r, t) weighs token t for the r-th part of the group's heads; the weights go through LDS, as
// bf16, into the A operand of V_MFMA_F32_16X16X16_BF16, one instruction for each of the lane's eight columns: after two V_PERM_B32 a lane
// holds one column of its four rows.  A tile's scores are requested before its rows (loads return in order), so that the weights are made while
// the rows arrive.  The weights, and the waves' factors when their sums meet, are 2^x as the hardware has it: what it flushes to zero is below
// 2^-126 of the largest.
//
// What bounds it is memory and, for that, bytes in flight: a CU has at most about 64 KB of misses on their way, so half of the CUs do not saturate
// the memory (128 of them: 4.5 TB/s of 6.5).  Hence 64 registers, tiles of 4 KB for each of 16 waves, and two workgroups to a CU, so that a row
// of the top-k and a run of values share one (8 sequences of 16384, 32 heads: values in 128 registers, alone on their CUs, 57 - 61 us
// for the launch, so 51; the values alone 49, the rows alone 14).
// Measured (us for the layer; one pass for scores and output, then the top-k -> so): 1 sequence, 32 heads, of 4096 21.7 -> 19.6, of 32768
// 50.1 -> 38.9; 8 of 16384 119.1 -> 115.5; 64 heads of 131072 144.6 -> 124.0.
struct ValueArgs {
    const float* P;
    int64_t ldp;
    float scale_log2e;
    float* part_acc;
    float* part_ml;
    uint16_t* out;
    int n_splits, chunk;      // runs per (sequence, KV head); chunk: a multiple of VALUE_WG_TILE tokens
    int wgs, pairs;           // workgroups that take them in turn; (sequence, KV head) pairs
    int g;                    // query heads per KV head
    int items;                // workgroups
    // V without a case distinction, which would cost the loop over runs registers: 16 rows start seq_step * b + head_step * kvh + group_step * n
    // from v, where n is their page, or the first one's token (paged: all bits, or none), and are row_bytes apart
    const uint16_t* v;
    const int32_t* seq_lens;
    const int32_t* table;     // [b][table_step]; not paged: an address that can be read, table_step 0
    int64_t seq_step, head_step, group_step;
    int G, table_step, paged;
    uint32_t row_bytes;
};
constexpr int VALUE_TILE = 16;
constexpr int VALUE_WG_TILE = VALUE_TILE * SEL_WAVES;
constexpr int VALUE_PAIRS_IN_ORDER = 64;
struct ValueLds {
    float m[SEL_WAVES][8], l[SEL_WAVES][8];
};
template <int GQ>
constexpr size_t value_lds_bytes() { return (size_t)SEL_WAVES * GQ * D * 4; }

template <int GQ>
__device__ __forceinline__ void weigh_values(const ValueArgs& a, int pair, int split, int L, int wave, float* sums_lds, ValueLds& st) {
    constexpr int TI = VALUE_TILE / 4;
    constexpr int HPL = GQ >= 4 ? GQ / 4 : 1;         // heads a lane weighs: those from head (row group % HROWS) * HPL on
    constexpr int HROWS = GQ / HPL;                   // row groups that weigh different heads
    const int kvh = pair % a.G, b = pair / a.G;
    const int64_t head0 = ((int64_t)b * a.G + kvh) * GQ;
    float* const wsum = sums_lds + wave * (GQ * D);   // [GQ][D], this wave's; before that its weights:
    __bf16* const wbuf = reinterpret_cast<__bf16*>(wsum);   // [head][row group][row load], the A operand's order
    int my_lane;                                      // (made here: not kept from run to run)
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(my_lane));
    const int begin = split * a.chunk;
    const int last = min(begin + a.chunk, L) - 1;
    const float* const prow = a.P + head0 * a.ldp;
    float m[HPL], l[HPL], p[HPL];
    f32x4 acc[8];                                     // column 8c + e; heads 4r .. 4r+3
#pragma unroll
    for (int j = 0; j < HPL; ++j) {
        m[j] = LOWEST;
        l[j] = 0.0f;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // A tile is 16 rows (a page): the address of its first row is uniform, a lane adds its row's distance from it, rows
    // past the end of the run that of its last token.
    u32x4 v[TI];
    const int32_t* const table = a.table + (int64_t)b * a.table_step;
    const uint16_t* const origin = a.v + ((int64_t)b * a.seq_step + (int64_t)kvh * a.head_step);
    int group = 0;                                    // page, or first token, of the tile to be requested next
    auto page_load = [&](int t_) {
        group = (uniform_load(table + ((min(t_, last) >> 4) & a.paged)) & a.paged) | (t_ & ~a.paged);
    };
    auto request_p = [&](int t_) {
        asm volatile("" : "+v"(my_lane));             // (no registers for what can be made of it)
        const uint32_t heads = (uint32_t)((my_lane >> 4) & (HROWS - 1)) * (uint32_t)(HPL * a.ldp);   // (32 bits: values_beside_topk)
        const uint32_t at = 4u * (heads + (uint32_t)min(t_ + (my_lane & 15), last));
#pragma unroll
        for (int j = 0; j < HPL; ++j) {
            uint64_t base = reinterpret_cast<uint64_t>(prow + j * a.ldp);
            asm volatile("" : "+s"(base));            // (scalar base and 32-bit distance: no 64-bit sums in vector registers)
            p[j] = *reinterpret_cast<const __attribute__((address_space(1))) float*>(reinterpret_cast<const __attribute__((address_space(1))) char*>(base) + at);
        }
    };
    auto request_v = [&](int t_) {
        asm volatile("" : "+v"(my_lane));
        const int rows = last - t_;
        const char* const at = reinterpret_cast<const char*>(origin + (int64_t)group * a.group_step);
#pragma unroll
        for (int i = 0; i < TI; ++i)
            v[i] = stream_load(reinterpret_cast<const uint16_t*>(at + ((uint32_t)min(i * 4 + (my_lane >> 4), rows) * a.row_bytes + 16u * (uint32_t)(my_lane & 15))));
    };
    int t0 = begin + wave * VALUE_TILE;
    page_load(t0);
    if (t0 <= last) {
        request_p(t0);
        request_v(t0);
        page_load(t0 + VALUE_WG_TILE);
    }
    for (; t0 <= last; t0 += VALUE_WG_TILE) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : "+v"(my_lane));
        // lane (r, t) weighs token t; token t is row load t / 4 of row group t % 4
        const int t = my_lane & 15, r = my_lane >> 4;
        __bf16* const put = wbuf + (r & (HROWS - 1)) * (HPL * VALUE_TILE) + (t & 3) * TI + (t >> 2);
        float corr[HPL];
        bool same = true;
#pragma unroll
        for (int j = 0; j < HPL; ++j) {
            const float z = t0 + t <= last ? p[j] * a.scale_log2e : -INFINITY;
            const float m_new = fmaxf(m[j], row_max16(z));
            corr[j] = __builtin_amdgcn_exp2f(m[j] - m_new);
            same = same && __ballot(m_new != m[j]) == 0;
            m[j] = m_new;
            // the weight enters numerator and denominator as the same bf16 value
            const __bf16 pb = (__bf16)__builtin_amdgcn_exp2f(z - m_new);
            put[j * VALUE_TILE] = pb;                 // (row groups that repeat a head's weights write the same)
            l[j] = l[j] * corr[j] + (float)pb;
        }
        const bool more = t0 + VALUE_WG_TILE <= last;
        // ahead of the rows: the weights are made while these arrive (a group of 8 has no registers for that so early)
        if (GQ < 8 && more) request_p(t0 + VALUE_WG_TILE);
        if (!same) {                                  // uniform; rare after the first tiles
#pragma unroll
            for (int hh = 0; hh < (GQ < 4 ? GQ : 4); ++hh) {
                // head 4r + hh: its factor is with the lanes that weigh it
                const float f0 = lane_value(corr[hh % HPL], (hh / HPL) * 16);
                const float f1 = GQ == 8 ? lane_value(corr[hh % HPL], (hh / HPL) * 16 + 32) : f0;
                const float g = r & 1 ? f1 : f0;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e][hh] *= g;
            }
        }
        wave_lds_sync();
        // rows of A beyond the group repeat its heads
        const s16x4 wa = *reinterpret_cast<const s16x4*>(wbuf + (my_lane & (GQ - 1)) * VALUE_TILE + r * TI);
        // the same column of the lane's four rows
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t pick = e & 1 ? 0x07060302u : 0x05040100u;
            const uint2 col = make_uint2(__builtin_amdgcn_perm(v[1][e >> 1], v[0][e >> 1], pick), __builtin_amdgcn_perm(v[3][e >> 1], v[2][e >> 1], pick));
            acc[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wa, __builtin_bit_cast(s16x4, col), acc[e], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            if (GQ >= 8) request_p(t0 + VALUE_WG_TILE);
            request_v(t0 + VALUE_WG_TILE);
            page_load(t0 + 2 * VALUE_WG_TILE);
        }
        wave_lds_sync();                              // the weights are rewritten next time
    }
    asm volatile("" : "+v"(my_lane));
    const int tid = wave * 64 + my_lane;
    // The waves' sums meet in LDS: lanes of row group r hold heads 4r .. 4r+3.
    {
        const int r = (tid >> 4) & 3, c = tid & 15;
        if (4 * r < GQ) {
#pragma unroll
            for (int hh = 0; hh < (GQ < 4 ? GQ : 4); ++hh) {
                float* const dst = wsum + (4 * r + hh) * D + c * 8;
                *reinterpret_cast<f32x4*>(dst) = f32x4{acc[0][hh], acc[1][hh], acc[2][hh], acc[3][hh]};
                *reinterpret_cast<f32x4*>(dst + 4) = f32x4{acc[4][hh], acc[5][hh], acc[6][hh], acc[7][hh]};
            }
        }
    }
#pragma unroll
    for (int j = 0; j < HPL; ++j) {
        const float ls = row_sum16(l[j]);
        const int r = (tid >> 4) & 3;
        if ((tid & 15) == 0 && r < HROWS) {
            st.m[wave][r * HPL + j] = m[j];
            st.l[wave][r * HPL + j] = ls;
        }
    }
    __syncthreads();
    for (int o = tid; o < GQ * D; o += SEL_THREADS) {
        const int h = o / D, col = o % D;
        float M = st.m[0][h];
#pragma unroll
        for (int wv = 1; wv < SEL_WAVES; ++wv) M = fmaxf(M, st.m[wv][h]);
        float A = 0.0f, Ls = 0.0f;
#pragma unroll 4
        for (int wv = 0; wv < SEL_WAVES; ++wv) {
            const float f = __builtin_amdgcn_exp2f(st.m[wv][h] - M);
            A = __builtin_fmaf(sums_lds[wv * (GQ * D) + o], f, A);
            Ls = __builtin_fmaf(st.l[wv][h], f, Ls);
        }
        if (L <= a.chunk) {                           // this workgroup saw all tokens
            a.out[(head0 + h) * D + col] = f32_to_bf16_rne(Ls > 0.0f ? A / Ls : 0.0f);
        } else {
            const int64_t p_ = (head0 + h) * a.n_splits + split;
            a.part_acc[p_ * D + col] = A;
            if (col == 0) {
                a.part_ml[p_ * 2] = M;
                a.part_ml[p_ * 2 + 1] = Ls;
            }
        }
    }
}

// The top-k over whole rows and the values in one launch, 1-D grid of n_topk + va.items workgroups.  Workgroup i of the values takes the runs
// i / pairs, i / pairs + wgs, ... of pair i % pairs: where sequences are shorter than the bound, the workgroups with work come first.  Of few pairs the
// runs of one come together, if a workgroup has no more than one of them (us for the layer, first runs first and so: 8 pairs of 131072, groups of 8, 125.5
// and 119.7; 64 of 16384 110.3 and 108.4; 16 of 131072, paged, 211.3 and 209.0; 32 of 16384, paged, 62.1 and 62.3; 128 of 9000, paged, 123.9 and 124.5; 256 of
// 8192 206.2 and 207.5). Rows and runs take turns of 256, a
// workgroup for every CU (where there are as many), what is left of either comes at the end: the dispatcher hands out workgroups strictly in order
// and in turn to the shader engines, so with a shorter turn all rows meet in a few engines and what follows them waits for a place elsewhere
// (turns of 8: 120 CUs idle for 18 of 64 us).
template <int ITEMS, int MTOP, bool GROUP8>
__global__ __launch_bounds__(SEL_THREADS, topk_lean(ITEMS, MTOP) ? 8 : 4) void topk_values_kernel(const float* __restrict__ P, int64_t ldp,
                                                                      const int32_t* __restrict__ seq_lens,
                                                                      int32_t* __restrict__ rho_head, int H, int k, int budget,
                                                                      int window, int n_sink, int B, ValueArgs va) {
    extern __shared__ uint64_t sort_buf[];
    const int n_topk = H * B, x = blockIdx.x, turns = min(n_topk, va.items) / 256 * 256;
    int i = x - turns;                                // past the alternating part: first the rest of the one, then of the other kind
    bool values = i >= n_topk;
    if (x < 2 * turns) {
        values = (x >> 8) & 1;
        i = (x >> 9) * 256 + (x & 255);
    } else if (values) {
        i -= n_topk - turns;
    }
    if (!values) {
        topk_row<ITEMS, MTOP, false>(i % H, i / H, 0, B, P, ldp, seq_lens, rho_head, H, k, budget, window, 0, n_sink, nullptr, 0, 1, nullptr,
                                     FilterState{}, SliceLists{});
        return;
    }
    __shared__ ValueLds st;
    float* const lds = reinterpret_cast<float*>(sort_buf);
    int wave = __builtin_amdgcn_readfirstlane(wave_id()), pair = i % va.pairs, first = i / va.pairs;
    if (va.wgs == va.n_splits && va.pairs <= VALUE_PAIRS_IN_ORDER) {
        pair = i / va.n_splits;
        first = (i + pair) % va.n_splits;             // short sequences' idle workgroups: spread over the XCDs
    }
    const int L = uniform_load(va.seq_lens + pair / va.G);
#pragma clang loop unroll(disable)
    for (int run = first; run * va.chunk < L; run += va.wgs) {
        asm volatile("" : "+s"(pair), "+s"(wave));    // (scalar registers: every run makes what it needs of them anew)
        if constexpr (GROUP8) {                       // (its registers are too few beside the other groups' code)
            weigh_values<8>(va, pair, run, L, wave, lds, st);
        } else {
            if (va.g == 4) weigh_values<4>(va, pair, run, L, wave, lds, st);   // uniform
            else if (va.g == 2) weigh_values<2>(va, pair, run, L, wave, lds, st);
            else weigh_values<1>(va, pair, run, L, wave, lds, st);
        }
        lds_barrier();                                // read, before the next run writes
    }
}

// Merge of the split-K partials of one (sequence, head) row whose sequence kept more than one workgroup
// busy.  256 threads (`tid`): thread (c4, sr) owns output columns 4*c4 .. 4*c4+3 and folds the splits sr, sr+8, ...
// into a running (m, l, a[4]) with 16-byte loads; the eight split-rows then meet in LDS and the result
// is written as bf16.  ALONE: the workgroup has this row only; otherwise `row` is uniform per wave, may lie past the last
// one, and all of the workgroup's rows meet the barrier.
template <bool ALONE>
__device__ __forceinline__ void reduce_row(const ReduceArgs& r, int row, int seq, int tid, ReduceLds& lds) {
    const int c4 = tid & 31, sr = tid >> 5;
    const bool have = ALONE || row < r.rows;
    if (!have) row = r.rows - 1;
    const int64_t base = (int64_t)row * r.stride_splits;
    constexpr int U = 4;
    // The first batch of partials is requested before the token count is known (any of the
    // stride_splits slots may be read); what lies beyond the active splits is dropped by select,
    // never by a multiplication, because those slots hold whatever was there before.
    f32x4 va[U];
    f32x2 vml[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int sv = sr + 8 * u;
        const int64_t p = base + (sv < r.stride_splits ? sv : 0);
        va[u] = *reinterpret_cast<const f32x4*>(&r.part_acc[p * D + c4 * 4]);
        vml[u] = *reinterpret_cast<const f32x2*>(&r.part_ml[p * 2]);
    }
    const int n_splits = attn_active_splits(min(r.n_tok[seq], r.n_clip), r.chunk);
    // keep the requests above the branch (the compiler would sink them behind it)
    asm volatile("" ::"s"(n_splits));
#pragma unroll
    for (int u = 0; u < U; ++u) asm volatile("" ::"v"(va[u]), "v"(vml[u]));
    const bool merge = have && n_splits > 1;             // otherwise the attention kernel wrote the result itself
    if (ALONE && !merge) return;
    float mo = -INFINITY, lo = 0.0f;
    f32x4 ao = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = sr; merge && s0 < n_splits; s0 += 8 * U) {
        if (s0 != sr) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int sv = s0 + 8 * u;
                const int64_t p = base + (sv < n_splits ? sv : s0);
                va[u] = *reinterpret_cast<const f32x4*>(&r.part_acc[p * D + c4 * 4]);
                vml[u] = *reinterpret_cast<const f32x2*>(&r.part_ml[p * 2]);
            }
        }
        float mu[U], lu[U];
        bool there[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            mu[u] = vml[u].x;
            lu[u] = vml[u].y;
            there[u] = s0 + 8 * u < n_splits;
        }
        fold_pieces<U>(va, mu, lu, there, mo, lo, ao);
    }
    *reinterpret_cast<f32x4*>(&lds.a[sr][c4 * 4]) = ao;
    if (c4 == 0) {
        lds.m[sr] = mo;
        lds.l[sr] = lo;
    }
    __syncthreads();
    if (merge && tid < D) {
        float A, Ls;
        const float M = meet_in_lds(lds.m, lds.l, [&](int j) { return lds.a[j][tid]; }, A, Ls);
        r.out[(int64_t)row * D + tid] = f32_to_bf16_rne(Ls > 0.0f ? A / Ls : 0.0f);
        if (r.lse && tid == 0) r.lse[row] = M + log2f(Ls);
    }
}

// The merge as a launch of its own: grid (H, B).  (Plain leading arguments arrive preloaded in SGPRs.)
__global__ __launch_bounds__(REDUCE_THREADS) void attn_reduce_kernel(const float* __restrict__ part_acc,
                                                           const float* __restrict__ part_ml,
                                                           uint16_t* __restrict__ out,
                                                           const int32_t* __restrict__ n_tok, int n_clip,
                                                           int stride_splits, int chunk, int H,
                                                           float* __restrict__ lse) {
    __shared__ ReduceLds lds;
    const ReduceArgs r = {part_acc, part_ml, out, n_tok, n_clip, stride_splits, chunk, lse, 0};
    reduce_row<true>(r, (int)(blockIdx.y * H + blockIdx.x), (int)blockIdx.y, (int)threadIdx.x, lds);
}

// Streaming-read probe (benchmark support): every thread folds 16-byte loads of a plain buffer,
// eight in flight per lane, consecutive lanes on consecutive addresses.  What this kernel reaches
// is the practical ceiling of a read-only pass on the machine, to set beside the nominal HBM peak.
constexpr int PROBE_THREADS = 256;
constexpr int PROBE_UNROLL = 8;

__global__ __launch_bounds__(PROBE_THREADS) void probe_stream_read_kernel(const u32x4* __restrict__ src, int64_t n_vec,
                                                                           uint32_t* __restrict__ sink) {
    const int64_t stride = (int64_t)gridDim.x * PROBE_THREADS;
    u32x4 fold = {0u, 0u, 0u, 0u};
    int64_t i = (int64_t)blockIdx.x * PROBE_THREADS + threadIdx.x;
    for (; i + (PROBE_UNROLL - 1) * stride < n_vec; i += PROBE_UNROLL * stride) {
        u32x4 v[PROBE_UNROLL];
#pragma unroll
        for (int u = 0; u < PROBE_UNROLL; ++u) v[u] = __builtin_nontemporal_load(&src[i + u * stride]);
#pragma unroll
        for (int u = 0; u < PROBE_UNROLL; ++u) fold ^= v[u];
    }
    for (; i < n_vec; i += stride) fold ^= __builtin_nontemporal_load(&src[i]);
    const uint32_t f = fold.x ^ fold.y ^ fold.z ^ fold.w;
    if (f == 0x9e3779b9u) *sink = f;                 // keeps the loads alive; practically never taken
}

// Traffic probes (benchmark support): the memory system's rate for the access patterns of the attention
// kernels, without their arithmetic.  A workgroup of four waves walks chunks of 32 tiles; a wave reads a
// tile of 32 KB with 32 streaming loads of 16 bytes per lane in flight (what K and V of 64 tokens are), then
//   PATTERN 0: nothing else (a plain streaming read in this shape);
//   PATTERN 1: nothing else -- but the tile is 128 rows of 256 bytes gathered from a region four times as
//              large: row 4 j + (hash(j) mod 4), ascending with irregular gaps like a sorted token list;
//   PATTERN 2: streams its tile and writes 1 KB of results as four runs of 256 bytes in rows far apart,
//              right away (what a scoring pass does that stores every tile's scores);
//   PATTERN 3: streams its tile and keeps the 1 KB in LDS; the workgroup writes the chunk's 32 KB in one
//              burst (four runs of 8 KB) when the chunk is done.
// dst takes the results of patterns 2 and 3: one float per 128 bytes read.
constexpr int PROBE_CHUNK_TILES = 32;

template <int PATTERN>
__global__ __launch_bounds__(256) void probe_traffic_kernel(const u32x4* __restrict__ src, float* __restrict__ dst,
                                                             int64_t n_chunks) {
    __shared__ f32x4 stage[PATTERN == 3 ? PROBE_CHUNK_TILES * 64 : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int64_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
        for (int j = 0; j < PROBE_CHUNK_TILES / 4; ++j) {
            const int64_t t = ch * PROBE_CHUNK_TILES + j * 4 + wave;   // tile
            u32x4 v[32];
            if (PATTERN == 1) {
#pragma unroll
                for (int i = 0; i < 32; ++i) {
                    const int64_t jrow = t * 128 + i * 4 + (lane >> 4);
                    const uint32_t hsh = (uint32_t)jrow * 2654435761u;
                    v[i] = __builtin_nontemporal_load(&src[(jrow * 4 + (hsh >> 30)) * 16 + (lane & 15)]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 32; ++i) v[i] = __builtin_nontemporal_load(&src[t * 2048 + i * 64 + lane]);
            }
            u32x4 f = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < 32; ++i) f ^= v[i];
            const f32x4 o = {(float)f.x, (float)f.y, (float)f.z, (float)f.w};
            if (PATTERN == 2) {
                const int64_t g = t >> 9, col = (t & 511) * 64 + lane;
#pragma unroll
                for (int h = 0; h < 4; ++h) dst[(g * 4 + h) * 32768 + col] = o[h];
            } else if (PATTERN == 3) {
                stage[(j * 4 + wave) * 64 + lane] = o;
            } else if (f.x == 0x9e3779b9u) {
                dst[0] = o[0];                           // keeps the loads alive; practically never taken
            }
        }
        if (PATTERN == 3) {
            __syncthreads();
            constexpr int PER = PROBE_CHUNK_TILES * 64 / 4;   // 16-byte words per run: four runs of 8 KB
            for (int i = threadIdx.x; i < PROBE_CHUNK_TILES * 64; i += 256) {
                const int q = i / PER, w = i % PER;
                f32x4* const p = reinterpret_cast<f32x4*>(dst) + ((ch / 16) * 4 + q) * (16 * (int64_t)PER) + (ch % 16) * PER + w;
                __builtin_nontemporal_store(stage[i], p);
            }
            __syncthreads();
        }
    }
}

// Attention recall (Eq. 3): the share of a head's softmax mass that falls on its token set.  With
// lse = log2 of the softmax denominator (scores scaled by sm_scale * log2 e) over the set and over
// all tokens, the ratio of the two denominators is 2^(lse_set - lse_all).
__global__ void recall_kernel(const float* __restrict__ lse_set, const float* __restrict__ lse_all,
                              float* __restrict__ recall, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) recall[i] = exp2f(lse_set[i] - lse_all[i]);
}

}  // namespace cusa

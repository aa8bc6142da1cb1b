// How the attention passes are cut into workgroups.  Plain host code, no HIP: the rules can be looked at without a GPU.
#pragma once

#include <algorithm>
#include <cstdint>

namespace cusa {

constexpr int ATTN_WAVES = 4;       // waves of a workgroup
// Longest run of tokens a workgroup of the scoring variant may own: its scores wait in LDS (32 KB)
// until the run is done.
constexpr int ATTN_SCORE_CHUNK_CAP = 2048;
constexpr int ATTN_SCORE_CHUNK_CAP_G8 = 1024;

constexpr int MAX_SPLITS = 256;
constexpr int CUS = 256;
constexpr int TARGET_WGS = 2 * CUS; // two resident workgroups per CU
constexpr int SINGLE_WGS = 192;     // (sequence, KV head) pairs from which one workgroup each is enough;
constexpr int SINGLE_WGS_PAGED = 256;   // the block table's extra round trip per tile wants more of them
constexpr int CHUNK_CAP = 2048;
constexpr int SPARSE_CAP = 4096;    // a token set has the same length for nearly all sequences: longer single pieces stay in step
constexpr int PIECE = 1280;         // tokens per workgroup where the chip is filled a few times only
constexpr int MERGE_BATCH = 32;     // splits that the merge of partials asks for at a time
static_assert(ATTN_SCORE_CHUNK_CAP <= CHUNK_CAP && ATTN_SCORE_CHUNK_CAP_G8 <= CHUNK_CAP && ATTN_SCORE_CHUNK_CAP_G8 >= 1024 && PIECE >= 1024,
              "the split bound assumes it");

struct AttnPlan {
    int ti;        // row-load instructions per wave iteration (4 or 8; scoring variant 8 or 16)
    int chunk;     // tokens per workgroup, a multiple of the workgroup tile
    int n_splits;  // grid.x = ceil(n_max / chunk)
};

// Share of the resident slots that n workgroups keep busy over their rounds; a last round of at most one workgroup per CU
// takes about 0.6 of a round.
inline float round_share(int n) {
    const int last = n % TARGET_WGS;
    const float rounds = (float)(n / TARGET_WGS) + (last == 0 ? 0.0f : last <= TARGET_WGS / 2 ? 0.6f : 1.0f);
    return (float)n / (TARGET_WGS * rounds);
}

enum AttnKind { ATTN_FULL, ATTN_SPARSE, ATTN_SCORE };
inline int noalloc_splits(int n_max, int BG);

// Workgroup granularity for n_max tokens per (sequence, KV head).
// As many even pieces as keep all workgroups resident at once (TARGET_WGS / BG, rounded down: rounded up, the last piece
// is a stump and the workgroups no longer fit the chip in one go: 80 pairs of 4096 tokens 39.1 -> 33.9 us, 96 of 5000
// 51.9 -> 44.2).  From SINGLE_WGS pairs on a piece per pair: what it loses in balance it gains in the merge
// that falls away (224 pairs of 1024: two pieces 26.3, one 23.0 us; 472 of 832: 42 and 36).
// Where that leaves many slots idle (192 pairs: two pieces, 384 workgroups), a pass over all tokens takes more pieces that
// fill a round and a half (192 pairs of 3400: two pieces 63.6, three 64.7, four 59.0 us); with sparse attention's short
// lists it does not pay.
// Splits beyond MERGE_BATCH cost the merge a second round trip (8 pairs of 20000: 64 splits 19.1, 32 18.4 us), so few pairs are
// cut into MERGE_BATCH pieces while these stay short of 1536 tokens.
// Lists too long for one piece per workgroup (CHUNK_CAP) fill the chip more than once: pieces of CHUNK_CAP tokens, or
// of about PIECE where these make fewer than four rounds of workgroups, so that the last ones to finish -- of
// ragged lengths above all -- hold up less (128 pairs of 601 to 16383 tokens: pieces of 2048 106.3 us, of 1280 96.7; 376 of 2597 to
// 5195: 148.2 and 142.9; but 176 of 27576: 405.6 and 421.6).
// The scoring variant keeps its scores in LDS, hence its own caps, and writes them in bursts, which are
// better longer (pieces of 2048 against 1024 at 64 pairs of 16384: 121.3 and 123.7 us).
// Sparse attention takes one piece of up to SPARSE_CAP tokens (128 sequences of 8 KV heads, lists of 2560: 201 us, cut at 2048 249), but two where
// a few pairs are left over after every CU has had one, two, ... of the others and those long pieces would run alone (264 pairs of 4096: 118 us,
// in two pieces 105; 520: 198 and 184; 520 paged: 215 and 192; 384, half a round left over: 128 and 126; from three rounds
// on it no longer pays: 776 of 2560 172 and 172, of 4096 271 and 268).  It is never cut into more pieces than
// noalloc_splits says.
// Workgroups whose run is 512 tokens or longer load 8 rows per lane and iteration, which keeps more bytes in flight
// (304 pairs of 512, paged: 23.9 -> 20.0 us); shorter runs are faster with 4.
inline AttnPlan plan_attn(int n_max, int BG, int g, AttnKind kind, bool paged) {
    AttnPlan pl;
    const bool wide = kind == ATTN_SCORE;
    const int cap = kind == ATTN_FULL ? CHUNK_CAP : kind == ATTN_SPARSE ? SPARSE_CAP : g >= 8 ? ATTN_SCORE_CHUNK_CAP_G8 : ATTN_SCORE_CHUNK_CAP;
    int pieces = BG >= (paged ? SINGLE_WGS_PAGED : SINGLE_WGS) ? 1 : TARGET_WGS / BG;
    if (kind != ATTN_SPARSE && pieces > 1) {
        for (int more = pieces + 1; more * BG <= 2 * TARGET_WGS && n_max >= more * 512; ++more)
            if (round_share(more * BG) > round_share(pieces * BG) + 0.05f) pieces = more;
    }
    if (kind == ATTN_SPARSE && pieces == 1 && BG > CUS && BG < 3 * CUS && BG % CUS > 0 && BG % CUS < CUS / 2 && n_max >= CHUNK_CAP)
        pieces = std::min(2, noalloc_splits(n_max, BG));
    if (!wide && pieces > MERGE_BATCH && n_max <= MERGE_BATCH * 1536) pieces = MERGE_BATCH;
    int64_t chunk = ((int64_t)n_max + pieces - 1) / pieces;
    if (chunk > cap) {
        const bool few = (int64_t)((n_max + CHUNK_CAP - 1) / CHUNK_CAP) * BG < 4 * TARGET_WGS;
        const int piece = kind == ATTN_SCORE ? cap : kind == ATTN_FULL && few ? PIECE : CHUNK_CAP;
        pieces = (n_max + piece - 1) / piece;
        chunk = ((int64_t)n_max + pieces - 1) / pieces;
    }
    pl.ti = wide ? (chunk >= 512 ? 16 : 8) : chunk >= 512 ? 8 : 4;
    const int wg_tile = pl.ti * 4 * ATTN_WAVES;
    // whole tiles; the scoring variant's are large, so short runs go to the nearest (88 pairs of 743: 128 against 256 tokens)
    chunk = wide && chunk < 512 && chunk > wg_tile ? (chunk + wg_tile / 2) / wg_tile * wg_tile : (chunk + wg_tile - 1) / wg_tile * wg_tile;
    if ((n_max + chunk - 1) / chunk > MAX_SPLITS) {
        chunk = ((int64_t)n_max + MAX_SPLITS - 1) / MAX_SPLITS;
        chunk = (chunk + wg_tile - 1) / wg_tile * wg_tile;
    }
    pl.chunk = (int)chunk;
    pl.n_splits = (int)((n_max + chunk - 1) / chunk);
    if (pl.n_splits < 1) pl.n_splits = 1;
    return pl;
}

// Upper bound of plan_attn(m, BG', ...).n_splits over every m <= n_max and BG' >= BG: a token list is cut into
// TARGET_WGS / BG pieces (a scoring run rounded down to the nearest tile: at most half as many again), or up to twice as
// many and one if they have 512 tokens, or into pieces of at least 1024 tokens.  Monotone in n_max, so a workspace sized for a capacity serves every shorter bound.
inline int max_splits_bound(int n_max, int BG) {
    const int by_wgs = BG < TARGET_WGS ? TARGET_WGS / BG : 1;
    const int by_piece = (n_max + 511) / 512 < 2 * by_wgs + 1 ? (n_max + 511) / 512 : std::max(2 * by_wgs + 1, (n_max + 1023) / 1024);
    const int m = by_wgs + (by_wgs + 1) / 2 > by_piece ? by_wgs + (by_wgs + 1) / 2 : by_piece;
    return m < MAX_SPLITS ? m : MAX_SPLITS;
}

// Splits that decide whether cusa_sparse_attn_noalloc takes a problem (a statement to callers: it does not
// follow the plan, which never makes more): pieces of about 1/TARGET_WGS of all tokens, 2048 at most.
inline int noalloc_splits(int n_max, int BG) {
    int64_t chunk = ((int64_t)n_max * BG + TARGET_WGS - 1) / TARGET_WGS;
    if (chunk > CHUNK_CAP) chunk = CHUNK_CAP;
    const int wg_tile = (chunk >= 1024 ? 8 : 4) * 4 * ATTN_WAVES;
    chunk = (chunk + wg_tile - 1) / wg_tile * wg_tile;
    const int64_t n = ((int64_t)n_max + chunk - 1) / chunk;
    return (int)(n < 1 ? 1 : n > MAX_SPLITS ? MAX_SPLITS : n);
}

}  // namespace cusa

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
constexpr int PIECE = 1280;         // tokens per workgroup of a ragged batch that fills the chip once or twice
constexpr int MERGE_BATCH = 32;     // splits that the merge of partials asks for at a time
static_assert(ATTN_SCORE_CHUNK_CAP <= CHUNK_CAP && ATTN_SCORE_CHUNK_CAP_G8 <= CHUNK_CAP && ATTN_SCORE_CHUNK_CAP_G8 >= 1024 && PIECE >= 1024,
              "the split bound assumes it");

struct AttnPlan {
    int ti;        // row-load instructions per wave iteration (4 or 8; scoring variant 8 or 16, tiles of 128 or 256 tokens)
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

// Whole tiles of the scoring variant.
inline int64_t score_tiles(int64_t tokens) { return tokens < 512 ? (tokens + 127) / 128 * 128 : (tokens + 255) / 256 * 256; }
constexpr int SCORE_START = 64;     // what a workgroup of it costs besides its tokens, in tokens

// Workgroup granularity for n_max tokens per (sequence, KV head).
// As many even pieces as keep all workgroups resident at once (TARGET_WGS / BG, rounded down: rounded up, the last
// piece is a stump and the workgroups no longer fit the chip in one go: 80 pairs of 4096 tokens 39.1 -> 33.9 us, 96 of
// 5000 51.9 -> 44.2).  From SINGLE_WGS pairs on a piece per pair: what it loses in balance it gains in the merge that
// falls away (224 pairs of 1024: two pieces 26.3, one 23.0 us; 472 of 832: 42 and 36).
// Where fewer pairs leave many slots idle (136 pairs: three pieces, 408 workgroups), a pass over all tokens takes more
// pieces that fill a round and a half or two (144 pairs of 5000, paged: three pieces 0.93 of the time that pieces of
// 1/512 of all tokens take, five 0.88; 192 paged pairs of 3400: two 0.99, three 1.02, four 0.93); with sparse
// attention's short lists it does not pay.
// Splits beyond MERGE_BATCH cost the merge a second round trip, so few pairs are cut into MERGE_BATCH pieces while
// these stay short of 1536 tokens (8 pairs, 64 splits and 32, us: of 16384 15.2 and 13.8, 20000 17.1 and 15.9, 32768
// 25.1 and 24.0, 49152 34.8 and 33.8).
// Lists too long for one piece per workgroup (CHUNK_CAP) take even pieces of about 1/512 of all tokens, CHUNK_CAP at
// most.  A paged cache's sequences are of all lengths as a rule, and many workgroups have nothing to do: where pieces
// of CHUNK_CAP would fill the chip once or twice if all were of the full length, pieces of about PIECE hold up less at
// the end.  Mean over 4 draws of lengths and 12 sizes, against pieces of CHUNK_CAP: lengths L / 16, L / 4 or L / 2 to L
// 0.955 of the time (1024 tokens: 0.95, 1536: 0.98), all of length L 1.02; between two and four rounds 0.99 and 1.01,
// where a draw differs by more than that.  (128 pairs of 601 to 16383 tokens: 106.3 us, 97.3, in pieces of 1024 99.6.)
// A contiguous cache holds sequences of one length as a rule: 224 pairs of 6000 tokens, pieces of 2048 107.3 us, of
// 1280 114.6; 40 of 32768: 105.5 and 114.8.
// The scoring variant keeps its scores in LDS, hence its own caps, writes them in bursts, which are better longer
// (pieces of 2048 against 1024 at 64 pairs of 16384: 121.3 and 123.7 us), and its tiles are large (128 or 256 tokens):
// it takes 1/512 of all tokens, rounded up to whole tiles.  Even pieces as above, rounded to the nearest tile, were 2
// per cent slower over 177 selection layers of 8 to 512 pairs of 600 to 40000 tokens, and often by a last round with
// next to nothing in it (40 pairs of 5000 29.3 us, so 22.9; 24 of 9000 30.7 and 23.6; 128 of 1700 30.5 and 23.9; 256 of
// 1300 37.7 and 34.0).  Where the last of these pieces would open a second round of workgroups, somewhat longer ones
// that need one round are taken instead (104 pairs of 5000: 58.8 -> 50.6 us; 160 of 4000 68.4 -> 62.9; 320 of 700 34.3
// -> 26.4, which also saves the merge; not where they would be half as long again: 192 of 2600 52.4 -> 55.0).
// Sparse attention takes one piece of up to SPARSE_CAP tokens (128 sequences of 8 KV heads, lists of 2560: 201 us, cut
// at 2048 249), but two where a few pairs are left over after every CU has had one, two, ... of the others and those
// long pieces would run alone (264 pairs of 4096: 118 us, in two pieces 105; 520: 198 and 184; 520 paged: 215 and 192;
// 384, half a round left over: 128 and 126; from three rounds on it no longer pays: 776 of 2560 172 and 172, of 4096
// 271 and 268).  It is never cut into more pieces than noalloc_splits says.
// Workgroups whose run is 512 tokens or longer load 8 rows per lane and iteration, which keeps more bytes in flight
// (304 pairs of 512, paged: 23.9 -> 20.0 us); shorter runs are faster with 4.
inline AttnPlan plan_attn(int n_max, int BG, int g, AttnKind kind, bool paged) {
    AttnPlan pl;
    int64_t chunk = ((int64_t)n_max * BG + TARGET_WGS - 1) / TARGET_WGS;
    if (kind == ATTN_SCORE) {
        const int64_t cap = g >= 8 ? ATTN_SCORE_CHUNK_CAP_G8 : ATTN_SCORE_CHUNK_CAP;
        chunk = std::min(chunk, cap);
        pl.ti = chunk >= 512 ? 16 : 8;
        chunk = score_tiles(chunk);
        if ((n_max + chunk - 1) / chunk * BG > TARGET_WGS) {
            int64_t longer = score_tiles(chunk + 1);
            while (longer <= cap && (n_max + longer - 1) / longer * BG > TARGET_WGS) longer = score_tiles(longer + 1);
            const int64_t tokens = std::min(longer, (int64_t)n_max);
            if (longer <= cap && (tokens + SCORE_START) * 10 <= (chunk + SCORE_START) * (longer >= n_max ? 14 : 13)) {
                chunk = longer;
                pl.ti = chunk >= 512 ? 16 : 8;
            }
        }
    } else {
        const int even = (int)std::min((chunk + 127) / 128 * 128, (int64_t)CHUNK_CAP);
        int pieces = BG >= (paged ? SINGLE_WGS_PAGED : SINGLE_WGS) ? 1 : TARGET_WGS / BG;
        if (kind == ATTN_FULL && pieces > 1) {
            for (int more = pieces + 1; more * BG <= 2 * TARGET_WGS && n_max >= more * 512; ++more)
                if (round_share(more * BG) > round_share(pieces * BG) + 0.05f) pieces = more;
        }
        if (kind == ATTN_SPARSE && pieces == 1 && BG > CUS && BG < 3 * CUS && BG % CUS > 0 && BG % CUS < CUS / 2 && n_max >= CHUNK_CAP)
            pieces = std::min(2, noalloc_splits(n_max, BG));
        if (pieces > MERGE_BATCH && n_max <= MERGE_BATCH * 1536) pieces = MERGE_BATCH;
        chunk = ((int64_t)n_max + pieces - 1) / pieces;
        if (chunk > (kind == ATTN_SPARSE ? SPARSE_CAP : CHUNK_CAP)) {
            const int64_t wgs = (int64_t)((n_max + CHUNK_CAP - 1) / CHUNK_CAP) * BG;
            const bool ragged = kind == ATTN_FULL && paged && wgs > TARGET_WGS && wgs <= 2 * TARGET_WGS;
            const int piece = kind == ATTN_SPARSE ? CHUNK_CAP : ragged ? PIECE : even;
            pieces = (n_max + piece - 1) / piece;
            chunk = ((int64_t)n_max + pieces - 1) / pieces;
        }
        pl.ti = chunk >= 512 ? 8 : 4;
    }
    const int wg_tile = pl.ti * 4 * ATTN_WAVES;
    chunk = (chunk + wg_tile - 1) / wg_tile * wg_tile;
    if ((n_max + chunk - 1) / chunk > MAX_SPLITS) {
        chunk = ((int64_t)n_max + MAX_SPLITS - 1) / MAX_SPLITS;
        chunk = (chunk + wg_tile - 1) / wg_tile * wg_tile;
    }
    pl.chunk = (int)chunk;
    pl.n_splits = (int)((n_max + chunk - 1) / chunk);
    if (pl.n_splits < 1) pl.n_splits = 1;
    return pl;
}

// Workgroups per pair for n pieces each of BG pairs: about `limit` in all at most, all with as many pieces (some with one less).
inline int in_turn(int n, int BG, int limit) {
    const int64_t rounds = ((int64_t)n * BG + limit - 1) / limit;
    return (int)std::max<int64_t>(1, (n + rounds - 1) / rounds);
}

// Whether an attention launch merges its pieces itself (wait_and_merge) instead of leaving them to a second launch: where the host, 3 us a launch,
// takes longer than the GPU, that is where runs are short, and where the partial sums, written past the caches in twice the bytes, are few.
// rows: batch * query heads; in_step: one layer of several that are enqueued together, so that the GPU is behind the host.  (Launches captured into a
// graph, whose replay keeps no host waiting, always leave the merge to a second one: see MergeWords.)
// (Layer of one sequence, us, GPU alone / calls one after the other from Python, two launches and so: 32 heads, list of 1024, 512 rows of partial
// sums, 6.3 / 9.8 and 6.4 / 6.7; of 2048, 1024 rows, 6.9 / 9.8 and 6.9 / 6.7; all of 4096 tokens, 1024, 7.7 / 9.9 and 7.9 / 7.7; 64 heads, 1024, 1024
// rows, 6.9 and 7.85 / 7.5, 4096, 2048 rows, 8.4 / 9.7 and 9.2 / 9.3; 4 sequences, 512, 6.9 and 7.0 / 6.7.  Runs of 512 tokens: 8 sequences, lists of 4096, 26.2 and
// 27.1, the waiting costs more than a launch.)
// A merging workgroup holds a place while it waits, two of them to a row.  A CU has room for two workgroups of the kernels for groups of 8 and for four of the
// others, an XCD of 32 CUs for 64 and 128: the waiting ones of three launches of 64 and of 128 rows, 16 and 32 of each launch on an XCD, leave a fourth launch's pieces
// places there.  (Where they do not -- launches of both kinds, more queues, a stream bound to few CUs, other programs --, rows are handed over: wait_and_merge.)
constexpr int MERGE_ROWS_MAX = 128;
constexpr int MERGE_ROWS_MAX_G8 = 64;
constexpr int MERGE_RUN = 128;
constexpr int MERGE_PIECES_MAX = 1024;   // rows of partial sums
constexpr int MERGE_PIECES_STEP = 512;
inline bool merges_itself(const AttnPlan& pl, int64_t rows, int g, bool in_step) {
    return pl.ti == 4 && pl.n_splits > 1 && pl.chunk <= MERGE_RUN && rows <= (g >= 8 ? MERGE_ROWS_MAX_G8 : MERGE_ROWS_MAX) &&
           rows * pl.n_splits <= (in_step ? MERGE_PIECES_STEP : MERGE_PIECES_MAX);
}

// The pieces that a row's merge in the launch waits for: those that have tokens, and never more than the launch has (a length beyond the
// bound that the plan was made for must not make it wait for, or take, another row's).
constexpr int merged_pieces(int n, int chunk, int n_splits) {
    const int a = (n + chunk - 1) / chunk;
    return a < 1 ? 1 : a < n_splits ? a : n_splits;
}

// The scoring pass (score_kernel): a workgroup for every workgroup tile, of 256 tokens (128 where these would be too few to keep every
// CU busy twice over); there is no partial result to merge, so nothing bounds their number but the time that idle ones take: where the bound is
// far above the lengths, which are not known here, nearly all have nothing to do (64 sequences of 8 KV heads, no tile to be scored: 65536
// workgroups are gone after 20.5 us, 32768 after 10.7, 8192 after 4.0).  Beyond SCORE_WGS of them each takes several of a (sequence, KV
// head)'s tiles in turn (32 sequences of 4096, 64 heads, bound 1000000, cusa_select, us: a workgroup for every tile 418, at most 131072 125, 65536
// 115, 32768 110; 64 of 32768 and no more 974, 974, 975, 991).  The second chance of the filtered selection finds nothing to do as a rule
// and has at most about 8192 (31 sequences of 4119 to 16478, the heads of the short ones flagged: in runs of 2048 tokens 54 us, in turn 22).
struct ScorePlan {
    int ti;        // row-load instructions of a wave: tiles of 128 or 256 tokens
    int n_splits;  // workgroups per (sequence, KV head)
};
constexpr int SCORE_WGS = 65536;
inline ScorePlan plan_score(int n_max, int BG, bool second_chance) {
    const int ti = second_chance || (int64_t)n_max * BG > 256 * TARGET_WGS ? 16 : 8, tile = ti * 4 * ATTN_WAVES;
    const int tiles = (n_max + tile - 1) / tile;
    return {ti, second_chance ? std::min(tiles, std::max(8, 8192 / BG)) : in_turn(tiles, BG, SCORE_WGS)};
}

// A selection layer's values (weigh_values): workgroups of 16 waves.
struct ValuePlan {
    int chunk;     // tokens of a run, a multiple of the workgroup tile
    int n_splits;  // runs per (sequence, KV head)
    int wgs;       // workgroups that take them in turn
};
constexpr int VALUE_TOKENS = 256;   // a tile of 16 for each wave
// A workgroup of 16 waves that has nothing to do takes 2.6 ns of all CUs' time, one of four waves 0.3: beyond VALUE_WGS of them each takes several runs
// (us for the layer, a workgroup for every run and so: 64 sequences of 4096, 64 heads, bound 131072 506 and 318, one pass 338; 128 of 3000 888 and
// 547, 535; 32 of 4096, bound 1000000 644 and 192, 363.  64 of 9000 and no more 524; in 2048 workgroups 537, in 1024 552).
constexpr int VALUE_WGS = 4096;
// The runs of at most 1536 tokens -- two to six tiles for every wave -- that give every CU one workgroup.  Beside fewer rows of the top-k (rows: their
// number) than CUs, those CUs that a row starts on are left out, 64 at most (8 pairs of 9000 tokens, us for the layer: best of 256-token steps from
// 256 to 4096 22.9, so 23.0; of 16384 26.1 and 26.1; of 32768 36.0 and 36.0; of 131072 109.8 and 109.8; 16 of 16384 36.4 and 36.4).  More rows share all
// CUs with the runs anyway (64 pairs of 1562, groups of 4: runs for 192 CUs 27.7, for 256 26.1; of 3125 36.5 and 34.9; of 5156 48.8 and 43.9).
// Where that would make longer runs or leave CUs without, many short runs that fill the CUs as they become free: of 768 tokens in layers of up to half
// a million, of 1024 in larger ones (over 150 layers of 32 to 128 pairs and 280000 to 1000000 tokens, runs of 512, 768, 1024, 1280, 1536, against the
// one pass: 0.964, 0.956, 0.963, 0.974, 0.980); of 1536 from 192 pairs on, which are one to three to a pair and have little left over (108 layers of 192
// to 512 pairs of 1560 to 3300, runs of 512 to 2048: 0.919, 0.919, 0.914, 0.911, 0.904, 0.915; 256 pairs of 2031, groups of 2: 1024 1.06, 1536 0.99).
inline ValuePlan plan_values(int n_max, int BG, int rows) {
    const int64_t tokens = (int64_t)n_max * BG;
    const int per_pair = CUS / BG;
    int64_t chunk = 1536 + 1;
    if (rows < CUS) chunk = (tokens + CUS - std::min(rows, 64) - 1) / (CUS - std::min(rows, 64));
    else if (per_pair * BG >= CUS - 32) chunk = ((int64_t)n_max + per_pair - 1) / per_pair;
    if (chunk > 1536) chunk = BG >= 192 ? 1536 : tokens < 1 << 19 ? 768 : 1024;
    chunk = std::max((chunk + VALUE_TOKENS - 1) / VALUE_TOKENS * VALUE_TOKENS, (int64_t)512);
    if ((n_max + chunk - 1) / chunk > MAX_SPLITS) {
        chunk = ((int64_t)n_max + MAX_SPLITS - 1) / MAX_SPLITS;
        chunk = (chunk + VALUE_TOKENS - 1) / VALUE_TOKENS * VALUE_TOKENS;
    }
    const int n = (int)std::max<int64_t>(1, (n_max + chunk - 1) / chunk);
    return {(int)chunk, n, in_turn(n, BG, VALUE_WGS)};
}

// Whether a row of the workspace's scores has room for every token, not just the candidates: see values_beside_topk, which asks for it.  Once true
// it stays true for longer bounds, so a workspace laid out for a capacity serves every shorter bound, and rows stay under 3 / 2 of the candidates.
inline bool scores_of_all_tokens(int64_t rows, int k, int window, int max_seq_len) {
    return !(k > 4096 && rows > 192) && (int64_t)window * 3 <= max_seq_len;
}

// At most so many rows of the top-k are cut into slices where they are long and have a launch of their own (plan_filter_slices).
constexpr int MAX_SLICED_ROWS = 256;

// Whether a selection layer that is not filtered scores all tokens first and makes its output from those scores while the top-k runs (score_kernel,
// topk_values_kernel); otherwise one pass over K and V makes the output and writes the candidates' scores (attn_kernel's scoring variant).
// rows: batch * query heads.
inline bool values_beside_topk(int64_t rows, int BG, int k, int window, int max_seq_len, int64_t token_step) {
    const int64_t tokens = (int64_t)BG * max_seq_len;
    // the rows and runs are workgroups of 1024 threads of a one-dimensional launch: fewer than 2^32 threads
    if (rows + BG + VALUE_WGS >= 1 << 22) return false;
    // a lane's distance from the first row of its 16 fits 32 bits (elements between tokens; 0: paged)
    if (token_step > 1 << 26) return false;
    // A sort of more than 4096 picks needs 94 registers and 130 KB of LDS, and the runs in its launch, a workgroup to a CU with it, wait for the rows:
    // beside more than 192 rows the one pass and a launch of the rows are faster (us, K 8192, one pass and so: 8 sequences of 10000, 256 rows 93.6
    // and 103.8, of 16384 126.5 and 136.7, of 32000 226.4 and 226.9; 6 of 16384, 192 rows, 107.8 and 107.5; 4 82.3 and 75.3).
    // (scores_of_all_tokens)
    // Layers that large take long enough for the one pass to fill the chip as well, and read P once less (64 sequences of 32768, groups of 8: 1747 and
    // 1816, 16 of 65536 859 and 858, 64 of 9000 561 and 525).
    if (tokens >= 8 << 20) return false;
    // One workgroup ranks a row beside the values.  The longer it is, the less its sample says about so few picks: too many pass the threshold, and the
    // row is ranked the general way, five times as slowly, while rows that the top-k's own launch cuts into slices rarely are; and of one or two pairs
    // the values take less time than the row.  (1 to 32 pairs, groups of 1, 4, 8, 300 to 7680 picks, scores independent or correlated over 64 tokens,
    // against the one pass: geometric mean and worst of 100000 tokens 0.89 and 1.02, 131072 0.94 and 1.03, 150000 0.91 and 1.03, 180000 0.93 and 1.03,
    // 220000 0.94 and 1.11, 262144 0.99 and 1.63; from 360000 to 1048576, with samples of 4096 keys, 1.11 to 1.77 and 6.1.)
    if (rows <= MAX_SLICED_ROWS && max_seq_len - window > 3 * 65536) return false;
    // Groups of 8: the one pass, in runs of at most 1024 tokens, is at its best where these fill its 512 resident workgroups once, most of them
    // (64 pairs of 5625: 54.4 and 56.3; 128 of 3125 66.8 and 69.3; 48 of 6875 54.0 and 55.6; 48 of 5833 51.5 and 51.1, of 8333 61.4 and 58.5).
    if (rows == 8 * (int64_t)BG && BG >= 48 && BG < 192 && tokens >= 9 << 15 && tokens < 13 << 15) return false;
    // The scores of a window are written and read for the output alone: 4 g bytes for the 256 of a row.  From a third of the tokens on the one pass
    // is as fast (8 sequences of 16384, 8 KV heads, us, one pass and so, window 0.3, 0.4, 0.5, 0.9 of the tokens: groups of 4 106.7 and 103.7, 105.5 and
    // 104.1, 102.6 and 104.4, 99.1 and 104.5; of 8 117.4 and 117.1, 117.1 and 117.6, 112.8 and 117.0, 108.9 and 119.0).  (With at most
    // UNION_MAX_POSITIONS candidates this also keeps the score rows of a group's heads within 32 bits of each other.)
    return scores_of_all_tokens(rows, k, window, max_seq_len);
}

// Upper bound of plan_attn(m, BG', ...).n_splits over every m <= n_max and BG' >= BG: a token list is cut into
// TARGET_WGS / BG pieces, rounded up or down, or up to twice as many and one if they have 512 tokens, or into pieces of
// at least 1024 tokens.
// Monotone in n_max, so a workspace sized for a capacity serves every shorter bound.
inline int max_splits_bound(int n_max, int BG) {
    const int by_wgs = (TARGET_WGS + BG - 1) / BG;
    const int by_piece = (n_max + 511) / 512 < 2 * by_wgs + 1 ? (n_max + 511) / 512 : std::max(2 * by_wgs + 1, (n_max + 1023) / 1024);
    return std::min(std::max(by_wgs, by_piece), MAX_SPLITS);
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

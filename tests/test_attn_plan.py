"""The launch plan of the attention passes (csrc/attn_plan.hpp), compiled for the host and looked at without a GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2508_07101_amd import build as lib_build

CXX = shutil.which("g++") or shutil.which("c++")
pytestmark = pytest.mark.skipif(CXX is None, reason="no host compiler")


def run_checks(tmp_path, body):
    """Compiles `body` (uses plan(n, pairs, g, kind, paged); FAIL(...) prints a line) and returns what it printed."""
    src = tmp_path / "check.cpp"
    src.write_text(r'''
#include <cstdio>
#include "attn_plan.hpp"
#include "call_tag.hpp"
using namespace cusa;
static int fails = 0;
#define FAIL(...) do { if (++fails <= 20) { std::printf(__VA_ARGS__); std::printf("\n"); } } while (0)
static AttnPlan plan(int n, int pairs, int g, AttnKind kind, bool paged) { return plan_attn(n, pairs, g, kind, paged); }
[[maybe_unused]] static const AttnKind KINDS[] = {ATTN_FULL, ATTN_SPARSE, ATTN_SCORE};
[[maybe_unused]] static int cap_of(int g) { return g >= 8 ? ATTN_SCORE_CHUNK_CAP_G8 : ATTN_SCORE_CHUNK_CAP; }
[[maybe_unused]] static int step(int n) { return n < 3000 ? 1 + n / 100 : 1 + n / 37; }     // lengths to look at, odd ones among them
int main() {
''' + body + '\n    return 0;\n}\n')
    exe = tmp_path / "check"
    subprocess.check_call([CXX, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", lib_build.CSRC, "-o", str(exe), str(src)])
    return subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout


def test_splits_cover_the_list_and_stay_within_what_the_workspace_and_callers_are_told(tmp_path):
    """Every plan covers its list with whole tiles; its splits fit a workspace laid out for any longer bound and any
    smaller number of pairs (the per-head kernels count heads), and the static scratch's promise."""
    out = run_checks(tmp_path, r'''
    for (int pairs = 1; pairs <= 1100; pairs += pairs < 80 ? 1 : 7)
        for (int n = 1; n <= 140000; n += step(n))
            for (int g : {1, 8})
                for (AttnKind kind : KINDS)
                    for (bool paged : {false, true}) {
                        const AttnPlan p = plan(n, pairs, g, kind, paged);
                        const int tile = p.ti * 4 * ATTN_WAVES;
                        if (p.chunk % tile || (int64_t)p.chunk * p.n_splits < n || (p.n_splits > 1 && (int64_t)p.chunk * (p.n_splits - 1) >= n))
                            FAIL("%d pairs of %d: %d pieces of %d", pairs, n, p.n_splits, p.chunk);
                        if (kind == ATTN_SCORE && p.chunk > cap_of(g) && p.n_splits * 2 <= MAX_SPLITS) FAIL("scores of %d tokens at a time", p.chunk);
                        for (int fewer : {pairs, (pairs + 1) / 2, (pairs + 7) / 8})
                            if (p.n_splits > max_splits_bound(n, fewer)) FAIL("%d pairs of %d: %d splits, bound %d", pairs, n, p.n_splits, max_splits_bound(n, fewer));
                        if (kind == ATTN_SPARSE && p.n_splits > noalloc_splits(n, pairs)) FAIL("%d pairs of %d: %d splits, told %d", pairs, n, p.n_splits, noalloc_splits(n, pairs));
                    }
    for (int pairs = 1; pairs <= 1100; ++pairs)
        for (int n = 1, last = 0; n <= 1300000; n += step(n)) {
            if (max_splits_bound(n, pairs) < last) FAIL("the bound shrinks at %d pairs of %d", pairs, n);
            last = max_splits_bound(n, pairs);
        }
''')
    assert out == "", out


def test_sparse_lists_are_cut_where_a_few_pairs_are_left_over(tmp_path):
    """Long single pieces of a few pairs would run alone after all the others (264 pairs of 4096: 118 us against 105)."""
    out = run_checks(tmp_path, r'''
    for (int pairs = 1; pairs <= 1100; ++pairs)
        for (int n = 2048; n <= 4096; n += 61)
            for (bool paged : {false, true}) {
                const AttnPlan p = plan(n, pairs, 4, ATTN_SPARSE, paged);
                const bool left_over = (pairs > 256 && pairs < 384) || (pairs > 512 && pairs < 640);
                if (left_over && p.n_splits != std::min(2, noalloc_splits(n, pairs))) FAIL("%d pairs of %d: %d pieces", pairs, n, p.n_splits);
                if (pairs >= 384 && pairs <= 512 && p.n_splits != 1) FAIL("%d pairs of %d: %d pieces", pairs, n, p.n_splits);
            }
''')
    assert out == "", out


def test_long_lists_take_long_pieces_unless_the_batch_is_paged_and_fills_the_chip_once_or_twice(tmp_path):
    """Small pieces help ragged batches; sequences of one length lose up to 9 per cent by them."""
    out = run_checks(tmp_path, r'''
    for (int pairs = 1; pairs <= 1100; pairs += pairs < 300 ? 1 : 7)
        for (int n = 2049; n <= 140000; n += step(n))
            for (bool paged : {false, true}) {
                const AttnPlan p = plan(n, pairs, 4, ATTN_FULL, paged);
                const int pieces = pairs >= (paged ? 256 : 192) ? 1 : 512 / pairs;
                if ((n + 2 * pieces) / (2 * pieces + 1) <= 2048) continue;            // one resident round, or two
                const int64_t rounds_of_long_ones = (int64_t)((n + 2047) / 2048) * pairs;
                const int want = paged && rounds_of_long_ones > 512 && rounds_of_long_ones <= 1024 ? (n + 1279) / 1280 : (n + 2047) / 2048;
                if (p.n_splits > want && p.n_splits <= 128) FAIL("%d pairs of %d, paged %d: %d pieces, not %d", pairs, n, paged, p.n_splits, want);
            }
    if (plan(32768, 40, 4, ATTN_FULL, false).n_splits != 16) FAIL("40 pairs of 32768");
    if (plan(6000, 224, 4, ATTN_FULL, false).n_splits != 3) FAIL("224 pairs of 6000");
    if (plan(2500, 248, 4, ATTN_FULL, false).n_splits != 2) FAIL("248 pairs of 2500");
    if (plan(3400, 192, 4, ATTN_FULL, false).n_splits != 3) FAIL("192 pairs of 3400");
    if (plan(16383, 128, 4, ATTN_FULL, true).n_splits != 13) FAIL("128 paged pairs of 16383");
''')
    assert out == "", out


def test_scoring_passes_open_no_round_for_next_to_nothing(tmp_path):
    """Runs of about 1 / 512 of all tokens, in whole tiles; rounded to the nearest tile or cut evenly, these sizes took a second round
    of workgroups and up to 30 per cent longer.  (Whole tiles: up to 255 tokens more; a run that saves a round: 1.4 times that and a start.)"""
    out = run_checks(tmp_path, r'''
    const int sizes[][2] = {{40, 5000}, {24, 9000}, {128, 1700}, {256, 1300}, {104, 5000}, {160, 4000}, {320, 700}, {192, 832}, {128, 744}};
    for (const auto& s : sizes)
        for (bool paged : {false, true}) {
            const AttnPlan p = plan(s[1], s[0], 4, ATTN_SCORE, paged);
            if (s[0] * p.n_splits > TARGET_WGS) FAIL("%d pairs of %d: %d workgroups", s[0], s[1], s[0] * p.n_splits);
        }
    for (int pairs = 1; pairs <= 1100; pairs += pairs < 80 ? 1 : 7)
        for (int n = 1; n <= 140000; n += step(n))
            for (int g : {1, 8}) {
                const AttnPlan p = plan(n, pairs, g, ATTN_SCORE, false);
                const int64_t share = std::min((int64_t)cap_of(g), ((int64_t)n * pairs + TARGET_WGS - 1) / TARGET_WGS);
                if (p.n_splits * 2 <= MAX_SPLITS && (p.chunk < share || std::min(p.chunk, n) > (share + 256 + 64) * 14 / 10))
                    FAIL("%d pairs of %d: runs of %d", pairs, n, p.chunk);
            }
''')
    assert out == "", out


def test_selection_layer_runs_cover_the_tokens_and_fit_the_workspace(tmp_path):
    """Runs of the values: whole tiles, the list covered, no run empty; their partials fit a workspace laid out for any longer bound and
    any smaller number of pairs.  The scoring pass has a workgroup for every tile, the second chance no more than that; of neither, nor of the values,
    are there more than what the idle ones of sequences far below the bound may cost."""
    out = run_checks(tmp_path, r'''
    (void)plan;
    for (int pairs = 1; pairs <= 1100; pairs += pairs < 80 ? 1 : 7)
        for (int n = 1; n <= 1300000; n += step(n)) {
            for (int rows : {pairs, 2 * pairs, 8 * pairs}) {
                const ValuePlan v = plan_values(n, pairs, rows);
                if (v.chunk % VALUE_TOKENS || (int64_t)v.chunk * v.n_splits < n || (v.n_splits > 1 && (int64_t)v.chunk * (v.n_splits - 1) >= n))
                    FAIL("values of %d pairs of %d: %d runs of %d", pairs, n, v.n_splits, v.chunk);
                if (v.wgs < 1 || v.wgs > v.n_splits || v.wgs * (int64_t)pairs > VALUE_WGS + pairs || (v.n_splits * (int64_t)pairs <= VALUE_WGS && v.wgs != v.n_splits))
                    FAIL("values of %d pairs of %d: %d workgroups for %d runs", pairs, n, v.wgs, v.n_splits);
                for (int fewer : {pairs, (pairs + 1) / 2, (pairs + 7) / 8})
                    if (v.n_splits > max_splits_bound(n, fewer)) FAIL("values of %d pairs of %d: %d runs, bound %d", pairs, n, v.n_splits, max_splits_bound(n, fewer));
            }
            for (bool second : {false, true}) {
                const ScorePlan p = plan_score(n, pairs, second);
                const int tile = p.ti * 4 * ATTN_WAVES, tiles = (n + tile - 1) / tile;
                if ((p.ti != 8 && p.ti != 16) || p.n_splits < 1 || p.n_splits > tiles || (!second && tiles * (int64_t)pairs <= SCORE_WGS && p.n_splits != tiles))
                    FAIL("scores of %d pairs of %d: %d workgroups for %d tiles", pairs, n, p.n_splits, tiles);
                if (p.n_splits * (int64_t)pairs > SCORE_WGS + pairs) FAIL("scores of %d pairs of %d: %d workgroups", pairs, n, p.n_splits * pairs);
            }
        }
''')
    assert out == "", out


def test_the_selection_layers_values_stay_within_their_kernels_limits(tmp_path):
    """Where the values are made beside the top-k: fewer than 2^32 threads in the launch, rows of V and of scores within 32 bits of bytes of each
    other, room for every token's score; for all that the selection accepts (up to 1179648 candidates, windows of any length)."""
    out = run_checks(tmp_path, r'''
    (void)plan;
    const int MAX_POSITIONS = 1179648;
    long taken = 0;
    for (int pairs : {1, 2, 7, 64, 1000, 65535, 524280, 4000000})
        for (int g : {1, 2, 4, 8})
            for (int64_t cand = 1; cand <= MAX_POSITIONS; cand += cand < 3000 ? 97 : cand / 3)
                for (int64_t window : {(int64_t)0, cand / 8, cand / 3, cand / 2, cand, 5 * cand, (int64_t)134217728, (int64_t)160000000, (int64_t)2000000000})
                    for (int64_t step : {(int64_t)0, (int64_t)128, (int64_t)1 << 26, ((int64_t)1 << 26) + 8, (int64_t)1 << 31}) {
                        if (cand + window > 2147483647) continue;
                        const int n = (int)(cand + window);
                        const int64_t rows = (int64_t)pairs * g;
                        if (!values_beside_topk(rows, pairs, 512, (int)window, n, step)) continue;
                        ++taken;
                        const ValuePlan v = plan_values(n, pairs, (int)rows);
                        const int64_t ldp = ((int64_t)n + 63) / 64 * 64;
                        if ((rows + (int64_t)pairs * v.wgs) * 1024 >= (int64_t)1 << 32) FAIL("%d pairs of %d, groups of %d: threads", pairs, n, g);
                        if (((g - 1) * ldp + n) * 4 >= (int64_t)1 << 32) FAIL("%d tokens, groups of %d: scores", n, g);
                        if (step * 2 * 15 >= (int64_t)1 << 32) FAIL("%lld elements between tokens", (long long)step);
                        if (!scores_of_all_tokens(rows, 512, (int)window, n)) FAIL("no room for the scores of %d tokens", n);
                    }
    if (taken < 2000) FAIL("only %ld taken", taken);
    for (int window : {0, 100, 12345, 1000000})                  // a workspace for a capacity serves every shorter bound
        for (int n = window + 1; n < window + 1179648; n += step(n))
            if (scores_of_all_tokens(256, 5000, window, n) || (scores_of_all_tokens(256, 512, window, n) && !scores_of_all_tokens(256, 512, window, n + 1))) FAIL("window %d at %d", window, n);
''')
    assert out == "", out


def test_selection_layers_that_one_pass_serves_faster(tmp_path):
    """Where the former pass over K and V beats the two of the values: many picks to sort beside many rows, wide windows, the largest layers, few
    rows of more than 196608 candidates (sizes that were measured 4 to 10 per cent slower)."""
    out = run_checks(tmp_path, r'''
    (void)plan;
    struct { int rows, pairs, k, window, n; bool beside; } const sizes[] = {
        {256, 64, 8192, 0, 16384, false}, {512, 64, 7168, 1024, 10000, false}, {128, 32, 8192, 0, 16384, true}, {256, 64, 4096, 1024, 16384, true},
        {512, 64, 600, 8500, 16384, false}, {32, 8, 500, 1100, 3300, true}, {4096, 512, 1536, 512, 32768, false}, {4096, 512, 1536, 512, 9000, true},
        {512, 64, 768, 256, 5625, false}, {512, 64, 768, 256, 8125, true}, {256, 64, 768, 256, 5625, true}, {64, 8, 768, 256, 45000, true},
        {64, 8, 3072, 1024, 197632, true}, {64, 8, 3072, 1024, 197633, false}, {1, 1, 1792, 256, 1048576, false}, {320, 40, 1792, 256, 200000, true}};
    for (const auto& s : sizes)
        if (values_beside_topk(s.rows, s.pairs, s.k, s.window, s.n, 128) != s.beside) FAIL("%d rows, %d pairs of %d, k %d", s.rows, s.pairs, s.n, s.k);
''')
    assert out == "", out


def test_filtered_layers_take_the_wide_tile(tmp_path):
    """Layers of 8 Mi scores and more in groups of up to 4, which is what the filtered pass is for: runs in tiles of 256 tokens, whatever the window."""
    out = run_checks(tmp_path, r'''
    (void)plan;
    for (int64_t pairs = 1; pairs <= 65535; pairs += pairs < 80 ? 1 : pairs / 7)
        for (int g : {1, 2, 4})
            for (int64_t n = ((int64_t)8 << 20) / (pairs * g); n <= 4000000; n += n / 5 + 1)
                for (bool paged : {false, true}) {
                    if (n < 64) continue;
                    const AttnPlan p = plan_attn((int)n, (int)pairs, g, ATTN_SCORE, paged);
                    if (p.ti != 16 || p.chunk % 256) FAIL("%lld pairs of %lld, groups of %d: ti %d, runs of %d", (long long)pairs, (long long)n, g, p.ti, p.chunk);
                }
''')
    assert out == "", out


def test_launches_that_merge_their_pieces_themselves_have_few_short_ones(tmp_path):
    """Only tiles of 16 tokens hold the code for it, so the rule asks for them; runs of at most 128 tokens, at most 1024 rows of partial sums,
    512 in a step of several layers."""
    out = run_checks(tmp_path, r'''
    if (merges_itself({8, 128, 4}, 32, 4, false) || !merges_itself({4, 128, 4}, 32, 4, false)) FAIL("tiles of 32 tokens");
    long taken = 0;
    for (int pairs = 1; pairs <= 1100; ++pairs)
        for (int n = 1; n <= 9000; n += step(n))
            for (int g : {1, 2, 4, 8})
                for (AttnKind kind : {ATTN_FULL, ATTN_SPARSE})
                    for (bool paged : {false, true}) {
                        const AttnPlan p = plan(n, pairs, g, kind, paged);
                        const int64_t rows = (int64_t)pairs * g;
                        const bool call = merges_itself(p, rows, g, false), step_ = merges_itself(p, rows, g, true);
                        taken += call;
                        if (call && (p.ti != 4 || p.chunk > 128 || p.n_splits < 2 || rows > (g == 8 ? 64 : 128) || rows * p.n_splits > MERGE_PIECES_MAX))
                            FAIL("%d pairs of %d, groups of %d: %d pieces of %d", pairs, n, g, p.n_splits, p.chunk);
                        if (step_ && (!call || rows * p.n_splits > MERGE_PIECES_STEP)) FAIL("%d pairs of %d, groups of %d in a step", pairs, n, g);
                    }
    if (taken < 1000) FAIL("only %ld taken", taken);
''')
    assert out == "", out


def test_a_row_waits_for_no_more_pieces_than_the_launch_has(tmp_path):
    """Pieces with tokens, at least one; a length beyond the plan's bound (a caller's slip) stays within the row's own pieces."""
    out = run_checks(tmp_path, r'''
    (void)plan;
    for (int chunk : {64, 128})
        for (int n_splits : {2, 5, 32})
            for (int n = 0; n <= 3 * chunk * n_splits; ++n) {
                int with_tokens = 0;
                for (int s = 0; s < n_splits; ++s) with_tokens += s * chunk < n;
                if (merged_pieces(n, chunk, n_splits) != std::max(1, with_tokens)) FAIL("%d tokens in %d pieces of %d: %d", n, n_splits, chunk, merged_pieces(n, chunk, n_splits));
            }
''')
    assert out == "", out


def test_tags_differ_and_a_machine_without_random_numbers_is_no_exception(tmp_path):
    """A tag stands for one call; what makes the first must not throw through the C interface."""
    out = run_checks(tmp_path, r'''
    (void)plan;
    struct None { None() { throw 1; } uint32_t operator()() { return 0; } };
    struct Empty { uint32_t operator()() { throw 2; } };
    if (tag_start<None>() == 0 || tag_start<Empty>() == 0) FAIL("no start");
    uint64_t last = 0;
    for (int i = 0; i < 1000; ++i) {
        const uint64_t t = new_tag();
        if (t == 0 || t == last || (uint32_t)t == (uint32_t)last || t >> 32 == last >> 32) FAIL("tags %llx, %llx", (unsigned long long)last, (unsigned long long)t);
        last = t;
    }
''')
    assert out == "", out

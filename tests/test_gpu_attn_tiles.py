"""The attention passes at the edges of their tiles: lists that end inside, at and just behind a wave's tile, a workgroup's tile and a
piece, empty lists, outputs at addresses that take no wide store -- against softmax(q K^T / sqrt d) V in float64.

The tolerance is derived: a weight is rounded to bf16 (2^-9 of it), in the numerator as in the denominator, which makes at most 2^-8 of the
weighted mean of |v|; the output is rounded to bf16 (2^-9 of it); sums are binary32.
"""
import ctypes
import math

import pytest
import torch

from paper_2508_07101_amd import binding as cb

pytestmark = pytest.mark.gpu
DEV, D, G = "cuda", 128, 2
LENGTHS = (1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 511, 513, 1025, 2049)


def _cache(lens, layout, gen):
    n, B = max(lens), len(lens)
    k = torch.randn((B, G, n, D), generator=gen, device=DEV).bfloat16()
    v = torch.randn((B, G, n, D), generator=gen, device=DEV).bfloat16()
    seq_lens = torch.tensor(lens, dtype=torch.int32, device=DEV)
    if layout != "paged":
        if layout == "token_major":
            return k, v, cb.KvCache(k.transpose(1, 2).contiguous().transpose(1, 2), v.transpose(1, 2).contiguous().transpose(1, 2), seq_lens, n)
        return k, v, cb.KvCache(k, v, seq_lens, n)
    pages = (n + 15) // 16
    table = torch.randperm(B * pages, generator=gen, device=DEV).to(torch.int32).view(B, pages)

    def pool(x):
        x = torch.nn.functional.pad(x, (0, 0, 0, pages * 16 - n)).view(B, G, pages, 16, D).transpose(1, 2).reshape(B * pages, G, 16, D)
        p = torch.empty_like(x)
        p[table.flatten().long()] = x
        return p
    return k, v, cb.KvCache(pool(k), pool(v), seq_lens, n, table)


def _check(got, q, k, v, tokens, what):
    """One sequence: got and q [H][D], k and v [G][n][D]."""
    if len(tokens) == 0:
        assert (got == 0).all(), what
        return
    q64, g = q.cpu().double(), q.shape[0] // G
    for h in range(q.shape[0]):
        kk, vv = k[h // g, tokens].cpu().double(), v[h // g, tokens].cpu().double()
        p = torch.softmax(kk @ q64[h] / math.sqrt(D), 0)
        want, mean_abs = p @ vv, p @ vv.abs()
        err = (got[h].cpu().double() - want).abs()
        bad = err > 2.0 ** -9 * want.abs() + 2.0 ** -8 * mean_abs + 1e-5
        assert not bad.any(), f"{what}, head {h}: {err.max().item()}"


@pytest.mark.parametrize("g", [1, 2, 4, 8])
@pytest.mark.parametrize("layout", ["head_major", "token_major", "paged"])
@pytest.mark.parametrize("shift", [0, 1])                  # elements the outputs stand behind an aligned address
def test_lists_that_end_at_the_edges_of_tiles(g, layout, shift):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(100 * g + shift)
    lens, H = list(LENGTHS), G * g
    B, budget = len(lens), 700
    k, v, kv = _cache(lens, layout, gen)
    q = torch.randn((B, H, D), generator=gen, device=DEV).bfloat16()
    params = cb.make_params(B, H, G, budget, budget // 4)
    ws = cb.alloc_workspace(params, max(lens), DEV)
    out = torch.full((B * H * D + 8,), 7.0, dtype=torch.bfloat16, device=DEV)
    view = out[shift: shift + B * H * D].view(B, H, D)
    cb.full_attn(params, q, kv, view, ws)
    for b, n in enumerate(lens):
        _check(view[b], q[b], k[b], v[b], torch.arange(n, device=DEV), f"full, {n} tokens")
    # token lists of every length that fits, one of them empty
    counts = [min(n, budget) for n in lens]
    counts[-1], counts[-2] = 0, 257
    idx = torch.zeros((B, budget), dtype=torch.int32, device=DEV)
    for b, n in enumerate(counts):
        idx[b, :n] = torch.randperm(lens[b], generator=gen, device=DEV)[:n].sort().values.to(torch.int32)
    cnt = torch.tensor(counts, dtype=torch.int32, device=DEV)
    cb.sparse_attn(params, q, kv, idx, cnt, view, ws)
    for b, n in enumerate(counts):
        _check(view[b], q[b], k[b], v[b], idx[b, :n].long(), f"sparse, {n} of {lens[b]} tokens")
    assert (out[:shift] == 7.0).all() and (out[shift + B * H * D:] == 7.0).all(), "written beside the outputs"


@pytest.mark.parametrize("g", [1, 2, 4, 8])
@pytest.mark.parametrize("n", [60, 64, 250, 1000, 2050, 9000])
def test_few_sequences_in_pieces(g, n):
    """One sequence, cut into as many pieces as fill the chip: whole tiles, remainders, a single token in the last piece."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n + g)
    for length in (n, n + 1):
        k, v, kv = _cache([length], "head_major", gen)
        q = torch.randn((1, G * g, D), generator=gen, device=DEV).bfloat16()
        params = cb.make_params(1, G * g, G, length, length // 4)
        ws = cb.alloc_workspace(params, length, DEV)
        out = torch.empty_like(q)
        idx = torch.arange(length, dtype=torch.int32, device=DEV)[None]
        cb.full_attn(params, q, kv, out, ws)
        _check(out[0], q[0], k[0], v[0], torch.arange(length, device=DEV), f"full, {length} tokens")
        cb.sparse_attn(params, q, kv, idx, torch.tensor([length], dtype=torch.int32, device=DEV), out, ws)
        _check(out[0], q[0], k[0], v[0], torch.arange(length, device=DEV), f"sparse, {length} tokens")


@pytest.mark.parametrize("g", [1, 4, 8])
@pytest.mark.parametrize("n,b", [(40, 64), (600, 64), (9000, 24), (600, 1)])     # a tile, several waves, several pieces, pieces merged in the launch
@pytest.mark.parametrize("below", [126, 127, 130, 132])
def test_weights_far_below_the_largest_count_beside_large_values(g, n, b, below):
    """The first token's weight is 2^-below of the last one's (the others': nothing) and its values are 2^120, the only ones that are not
    zero: it makes the whole output, also where the weight is subnormal in binary32 and bf16.  Exact powers of two but for the rounding of
    scores (2^-23 of `below`, times ln 2), weight and output (2^-9 each)."""
    H = G * g
    k, v = (torch.zeros((b, G, n, D), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    k[:, :, 0, 0], k[:, :, 1:-1, 0], v[:, :, 0] = -below, -400.0, 2.0 ** 120
    q = torch.zeros((b, H, D), dtype=torch.bfloat16, device=DEV)
    q[..., 0] = 1.0
    kv = cb.KvCache(k, v, torch.full((b,), n, dtype=torch.int32, device=DEV), n)
    params = cb.make_params(b, H, G, n, n // 4, sm_scale=math.log(2.0))
    ws, out = cb.alloc_workspace(params, n, DEV), torch.empty_like(q)
    idx = torch.arange(n, dtype=torch.int32, device=DEV).repeat(b, 1)
    for what in ("full", "sparse"):
        if what == "full":
            cb.full_attn(params, q, kv, out, ws)
        elif n <= 8192:
            cb.sparse_attn(params, q, kv, idx, kv.seq_lens, out, ws)
        want = 2.0 ** (120 - below)
        err = ((out.double() - want).abs() / want).max().item()
        assert err <= 2.0 ** -7, f"{what}: {out.flatten()[0].item()}, not {want}"


def _layer(b, H, Gk, L, K, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    k = torch.randn((b, Gk, L, D), generator=gen, device=DEV).bfloat16()
    v = torch.randn((b, Gk, L, D), generator=gen, device=DEV).bfloat16()
    q = torch.randn((b, H, D), generator=gen, device=DEV).bfloat16()
    kv = cb.KvCache(k, v, torch.full((b,), L, dtype=torch.int32, device=DEV), L)
    idx = torch.stack([torch.randperm(L, generator=gen, device=DEV)[:K].sort().values for _ in range(b)]).to(torch.int32)
    return q, kv, idx, torch.full((b,), K, dtype=torch.int32, device=DEV), cb.make_params(b, H, Gk, K, K // 4)


def _two_launches(call):
    """Runs `call` from a graph: what is captured leaves the merge of its pieces to a second launch."""
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    graph.replay()
    torch.cuda.synchronize()


def _words(ws, rows):
    """The part of a workspace that only launches which merge their pieces themselves write (its last bytes)."""
    return ws[-min(rows * 32, 1024) * 1040:]


def _merges_itself(call, ws, rows):
    ws.fill_(85)
    call()
    return bool((_words(ws, rows) != 85).any())


# groups of 1, 2, 4 and 8, one and several sequences; rows of partial sums: 512, 1024, 176, 512, 1024, 1024, 1024
IN_LAUNCH = [(1, 32, 8, 4096, 1024), (1, 32, 8, 4096, 2048), (1, 8, 8, 3000, 300), (4, 8, 8, 1040, 1024), (2, 16, 8, 2100, 2048), (4, 32, 8, 520, 512),
             (2, 32, 4, 1030, 1024)]


@pytest.mark.parametrize("b,H,Gk,L,K", IN_LAUNCH)
def test_pieces_merged_in_the_launch_whatever_the_workspace_held(b, H, Gk, L, K):
    """The bits of the two launches, from a workspace of random words, of ones, of an earlier call's words or a selection's, in a decode step,
    without a workspace, and beside a graph that is replayed on the same workspace; lists of several lengths where there are several sequences."""
    q, kv, idx, cnt, params = _layer(b, H, Gk, L, K, 5)
    cnt -= torch.tensor([0, 65, K, K - 65][:b], dtype=torch.int32, device=DEV)
    ws = cb.alloc_workspace(params, L, DEV)
    want, want_full, full, got = (torch.empty_like(q) for _ in range(4))
    _two_launches(lambda: cb.sparse_attn(params, q, kv, idx, cnt, want, ws))
    _two_launches(lambda: cb.full_attn(params, q, kv, want_full, ws))
    assert _merges_itself(lambda: cb.sparse_attn(params, q, kv, idx, cnt, got, ws), ws, b * H)
    assert _merges_itself(lambda: cb.full_attn(params, q, kv, full, ws), ws, b * H) or L in (520, 1030)   # (more than 1024 rows)
    rho, n_rho = torch.zeros_like(idx), torch.zeros_like(cnt)
    for fill in ("random", "ones", "earlier", "earlier", "selection"):
        if fill == "random":
            ws.random_(0, 256)
        elif fill == "ones":
            ws.fill_(255)
        elif fill == "selection" and L > K:
            cb.select(params, q, kv, rho, n_rho, ws)
        got.zero_(), full.zero_()
        cb.sparse_attn(params, q, kv, idx, cnt, got, ws)
        assert torch.equal(got, want), f"sparse, workspace: {fill}"
        cb.full_attn(params, q, kv, full, ws)
        assert torch.equal(full, want_full), f"full, workspace: {fill}"
    got.zero_()
    cb.sparse_attn_noalloc(params, q, kv, idx, cnt, got)
    assert torch.equal(got, want)
    # a step of several layers, against its selection's own list
    outs = [torch.empty_like(q) for _ in range(3)]
    step = cb.DecodeStep(params, [cb.LAYER_SELECT, cb.LAYER_SPARSE, cb.LAYER_FULL], [q] * 3, [kv] * 3, outs, rho, n_rho, ws)
    step.run()
    cb.sparse_attn(params, q, kv, rho, n_rho, got, ws)
    assert torch.equal(outs[1], got) and torch.equal(outs[2], want_full)
    q2 = q.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cb.sparse_attn(params, q2, kv, idx, cnt, got, ws)
        cb.full_attn(params, q2, kv, full, ws)
    for rep in range(5):
        q2.copy_(torch.randn(q.shape, device=DEV).bfloat16())
        g.replay()
        torch.cuda.synchronize()
        now = (got.clone(), full.clone())
        if rep == 2:
            ws.random_(0, 256)
        cb.full_attn(params, q2, kv, full, ws)
        assert torch.equal(now[1], full), f"replay {rep}, full"
        cb.sparse_attn(params, q2, kv, idx, cnt, want, ws)
        assert torch.equal(now[0], want), f"replay {rep}, sparse"


@pytest.mark.parametrize("b,H,Gk,L,K", IN_LAUNCH)
def test_rows_handed_over_to_the_pieces(b, H, Gk, L, K):
    """Merging workgroups that look never, once or a few times before they hand their rows over: whoever merges then, the bits are those of the
    two launches, and no row is left out."""
    q, kv, idx, cnt, params = _layer(b, H, Gk, L, K, 6)
    cnt -= torch.tensor([0, 65, K, K - 65][:b], dtype=torch.int32, device=DEV)
    ws, want = cb.alloc_workspace(params, L, DEV), torch.empty_like(q)
    _two_launches(lambda: cb.sparse_attn(params, q, kv, idx, cnt, want, ws))
    lib, desc = cb.load(), kv.desc()
    vp = ctypes.c_void_p

    def call(out, looks):
        status = lib.cusa_test_sparse_attn_looks(ctypes.byref(params), vp(q.data_ptr()), ctypes.byref(desc), vp(idx.data_ptr()), vp(cnt.data_ptr()),
                                                 vp(out.data_ptr()), vp(ws.data_ptr()), ctypes.c_size_t(ws.numel()), vp(cb._stream()), looks)
        assert status == cb.OK
    first = torch.empty_like(q)
    assert _merges_itself(lambda: call(first, 0), ws, b * H)
    for looks in (0, 1, 2, 4, 8, 256):
        outs = [torch.full_like(q, 9.0) for _ in range(20)]
        for out in outs:                                   # one after the other, as fast as they come
            call(out, looks)
        assert all(torch.equal(o, want) for o in outs), f"{looks} looks"
    assert lib.cusa_test_sparse_attn_looks(ctypes.byref(params), vp(q.data_ptr()), ctypes.byref(desc), vp(idx.data_ptr()), vp(cnt.data_ptr()),
                                           vp(first.data_ptr()), vp(ws.data_ptr()), ctypes.c_size_t(ws.numel()), vp(cb._stream()), -1) == cb.ERR_INVALID_ARG


@pytest.mark.parametrize("g", [1, 4, 8])
def test_a_graph_replayed_with_other_lengths_and_counts(g):
    """What a replay finds in the workspace is the replay before's: lists and sequences that grow, shrink and become empty between replays,
    each against an eager call of the moment."""
    b, Gk, L, K = 2, 4, 1000, 400
    q, kv, idx, cnt, params = _layer(b, Gk * g, Gk, L, K, 21)
    ws, ws2 = cb.alloc_workspace(params, L, DEV), cb.alloc_workspace(params, L, DEV)
    out, full = torch.zeros_like(q), torch.zeros_like(q)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cb.sparse_attn(params, q, kv, idx, cnt, out, ws)
        cb.full_attn(params, q, kv, full, ws)
    for lens, counts in (((1000, 1000), (400, 400)), ((70, 999), (65, 400)), ((1000, 64), (400, 1)), ((513, 1000), (0, 400)), ((1000, 1000), (400, 129))):
        kv.seq_lens.copy_(torch.tensor(lens, dtype=torch.int32))
        cnt.copy_(torch.tensor(counts, dtype=torch.int32))
        q.copy_(torch.randn(q.shape, device=DEV).bfloat16())
        for i, n in enumerate(lens):
            idx[i] = torch.randint(0, n, (K,), device=DEV).to(torch.int32)
        out.fill_(3.0), full.fill_(3.0)
        graph.replay()
        torch.cuda.synchronize()
        now, now_full = torch.empty_like(q), torch.empty_like(q)
        cb.sparse_attn(params, q, kv, idx, cnt, now, ws2)
        cb.full_attn(params, q, kv, now_full, ws2)
        assert torch.equal(out, now) and torch.equal(full, now_full), f"lengths {lens}, counts {counts}"


def test_captured_launches_leave_the_merge_to_a_second_one():
    """A replay has the tag of the capture, so no launch in a graph may go by it: the room for the words stays as it was.  (A call writes there.)"""
    need = 1696000                                         # bytes of the workspace before that room
    q, kv, idx, cnt, _ = _layer(1, 32, 8, 4096, 1024, 4)
    params = cb.make_params(1, 32, 8, 1024, 256)
    ws, out = cb.alloc_workspace(params, 4096, DEV), torch.zeros_like(q)
    ws.fill_(77)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cb.sparse_attn(params, q, kv, idx, cnt, out, ws)
    graph.replay()
    torch.cuda.synchronize()
    assert (ws[need:] == 77).all() and (out != 0).any()
    cb.sparse_attn(params, q, kv, idx, cnt, out, ws)
    assert (ws[need:] != 77).any()


@pytest.mark.parametrize("b,H,Gk,L,K,W,need", [(1, 32, 8, 4096, 1024, 256, 1696000), (2, 16, 16, 3000, 512, 128, 708864)])
def test_a_workspace_without_room_for_the_words_is_taken(b, H, Gk, L, K, W, need):
    """What a launch that merges its pieces itself wants on top is no condition: with the bytes of the partial sums alone a second launch merges,
    to the same bits; with less the call is refused, as ever."""
    q, kv, idx, cnt, _ = _layer(b, H, Gk, L, K, 9)
    params = cb.make_params(b, H, Gk, K, W)
    ws = cb.alloc_workspace(params, L, DEV)
    assert ws.numel() > need
    outs = []
    for room in (ws, ws[:need], ws[:need + 256], ws[:ws.numel() - 256]):
        outs.append(torch.zeros_like(q))
        cb.sparse_attn(params, q, kv, idx, cnt, outs[-1], room)
    assert all(torch.equal(o, outs[0]) for o in outs)
    with pytest.raises(cb.CusaError) as err:
        cb.sparse_attn(params, q, kv, idx, cnt, outs[0], ws[:need - 1])
    assert err.value.status == cb.ERR_WORKSPACE_TOO_SMALL


def test_pieces_merged_in_launches_of_two_streams():
    """Each stream has a workspace of its own; the launches overlap as they like."""
    layers = [_layer(1, 32, 8, 4096, 1024, seed) for seed in (1, 2)]
    want = []
    for q, kv, idx, cnt, params in layers:
        out = torch.empty_like(q)
        cb.sparse_attn(params, q, kv, idx, cnt, out, cb.alloc_workspace(params, 4096, DEV))
        want.append(out)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in layers]
    wss = [cb.alloc_workspace(lay[4], 4096, DEV) for lay in layers]
    outs = [[torch.empty_like(lay[0]) for _ in range(50)] for lay in layers]
    torch.cuda.synchronize()
    for i in range(50):
        for s, lay, ws, out in zip(streams, layers, wss, outs):
            with torch.cuda.stream(s):
                cb.sparse_attn(lay[4], *lay[:4], out[i], ws)
    torch.cuda.synchronize()
    for w, out in zip(want, outs):
        assert all(torch.equal(o, w) for o in out)


@pytest.mark.parametrize("g", [1, 2, 4, 8])
@pytest.mark.parametrize("b,Gk,L,K", [(8, 8, 5000, 2048), (16, 8, 3000, 700), (8, 2, 5000, 2048), (1, 2, 300, 65)])
@pytest.mark.parametrize("per_head", [False, True])
def test_a_token_scores_the_same_in_passes_of_any_tile(g, b, Gk, L, K, per_head):
    """The recall of a set is a ratio of two passes, over the set and over all tokens, which take tiles of different widths.  Here scores reach
    2^20, where the last bit of a sum makes a factor of 2^0.1, and each head's largest lies by more than 2^8 above its others: its weight is 1, the
    others' are nothing.  If the sets hold the largest the recall is 1, and 2^0 exactly; otherwise it is 0."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(g + L)
    H = Gk * g
    k = torch.randn((b, Gk, L, D), generator=gen, device=DEV).bfloat16() * 1024
    q = torch.randn((b, H, D), generator=gen, device=DEV).bfloat16() * 1024
    kv = cb.KvCache(k, k, torch.full((b,), L, dtype=torch.int32, device=DEV), L)
    params = cb.make_params(b, H, Gk, K, K // 4)
    ws, recall = cb.alloc_workspace(params, L, DEV), torch.empty((b, H), dtype=torch.float32, device=DEV)
    scores = torch.stack([k[:, h // g].double() @ q[:, h].double()[..., None] for h in range(H)], 1)[..., 0] / math.sqrt(D)
    top = scores.topk(2)
    clear = top.values[..., 0] - top.values[..., 1] > 2.0 ** 8
    assert clear.float().mean() > 0.9
    lists = torch.rand((b, H if per_head else 1, L), generator=gen, device=DEV)
    held = torch.arange(H, device=DEV) % 3 > 0                 # heads whose sets hold their largest
    for h in range(H):
        lists[:, h if per_head else 0].scatter_(1, top.indices[:, h, :1], 2.0 if held[h] else -1.0)
    idx = lists.topk(K).indices.sort().values.to(torch.int32)
    want = (idx.view(b, -1, 1, K) == top.indices[:, :, :1, None].to(torch.int32)).any(-1).view(b, H).float()
    assert (want == 1).any() and (want == 0).any()
    cnt = torch.full((b,), K, dtype=torch.int32, device=DEV)
    cb.attention_recall(params, q, kv, idx if per_head else idx[:, 0].contiguous(), cnt, recall, ws, per_head=per_head)
    assert torch.equal(recall[clear], want[clear]), f"{(recall != want)[clear].sum().item()} of {clear.sum().item()}: {recall[clear & (recall != want)][:4].tolist()}"

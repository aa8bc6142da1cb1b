"""The top-k's own time on scores as attention has them: correlated along the sequence, or repeating.  The kernels' durations
come from the library's timing facility; they are compared with those of the same call on independent scores, on the
same device a moment earlier."""
import pytest
import torch

from paper_2508_07101_amd import binding as cb

pytestmark = pytest.mark.gpu
DEV, D, G = "cuda", 128, 8


def _topk_us(B, H, L, K, W, k, span=0, distinct=0, layer=False):
    """Fastest of five means of ten calls of cusa_select, or (layer) of a selection layer, whose values share the top-k's launch.
    span: each span of that many positions has an offset of its own, as wide as the scores are spread; distinct: that many
    different keys."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(11)
    q = torch.randn((B, H, D), generator=gen, device=DEV, dtype=torch.bfloat16)
    keys = torch.randn((B, G, distinct or L, D), generator=gen, device=DEV, dtype=torch.bfloat16)
    if distinct:
        keys = keys[:, :, torch.randint(distinct, (L,), generator=gen, device=DEV)].contiguous()
    if span:
        groups = q.float().view(B, G, -1, D)
        u = torch.nn.functional.normalize(groups.sum(2), dim=-1)          # moves the scores of all heads of a group alike
        per = (groups * u.unsqueeze(2)).sum(-1).mean(2, keepdim=True)
        off = torch.randn((B, G, (L + span - 1) // span), generator=gen, device=DEV) * D ** 0.5 / per
        keys = (keys.float() + off.repeat_interleave(span, 2)[:, :, :L].unsqueeze(-1) * u.unsqueeze(2)).to(torch.bfloat16)
    kv = cb.KvCache(keys, keys, torch.full((B,), L, dtype=torch.int32, device=DEV), L)
    p = cb.make_params(B, H, G, K, W, k)
    idx = torch.zeros((B, K), dtype=torch.int32, device=DEV)
    cnt = torch.zeros((B,), dtype=torch.int32, device=DEV)
    ws = cb.alloc_workspace(p, L, DEV)
    out = torch.empty_like(q)

    def call():
        if layer:
            cb.select_layer(p, q, kv, out, idx, cnt, ws)
        else:
            cb.select(p, q, kv, idx, cnt, ws)

    call()
    torch.cuda.synchronize()
    best = float("inf")
    cb.profile_enable(True)
    try:
        for _ in range(5):
            cb.profile_reset()
            for _ in range(10):
                call()
            prof = cb.profile_read()
            best = min(best, sum(v["total_ms"] for name, v in prof.items() if name.startswith("topk")) * 100.0)
    finally:
        cb.profile_enable(False)
        cb.profile_reset()
    return best


LAYER = pytest.mark.parametrize("layer", [False, True])
SIZES = [(1, 32, 32768, 2048, 512, 0), (8, 32, 16384, 4096, 1024, 0), (16, 32, 16384, 2048, 512, 0),
         (1, 64, 131072, 4096, 1024, 0)]


@LAYER
@pytest.mark.parametrize("size", SIZES)
def test_scores_correlated_along_the_sequence_take_no_longer(size, layer):
    """One list for the whole row: where its best candidates stand does not matter.  (With a sixteenth of the list for
    each wave these took 2.5 to 6 times as long as independent scores.)"""
    plain, clustered = _topk_us(*size, layer=layer), _topk_us(*size, span=256, layer=layer)
    print(f"[time] {'layer' if layer else 'select'} {size}: independent {plain:.1f} us, correlated {clustered:.1f} us", flush=True)
    assert clustered < 1.5 * plain


@LAYER
@pytest.mark.parametrize("size,span", [((1, 32, 30512, 2560, 512, 0), 256), ((1, 32, 30512, 2560, 512, 0), 64),
                                       ((1, 64, 131072, 2048, 512, 0), 64), ((1, 32, 60512, 2560, 512, 0), 64)])
def test_the_sample_speaks_for_rows_correlated_along_the_sequence(size, span, layer):
    """The threshold's sample is spread over the row in short runs and a second threshold goes by what the first let through.
    (Half the row in 256-key pieces, or 64-key runs, and twice as many the second time: 1.6 to 4 times as long.)"""
    plain, clustered = _topk_us(*size, layer=layer), _topk_us(*size, span=span, layer=layer)
    print(f"[time] {'layer' if layer else 'select'} {size} spans of {span}: independent {plain:.1f} us, correlated {clustered:.1f} us", flush=True)
    assert clustered < 1.4 * plain


@LAYER
@pytest.mark.parametrize("size", SIZES[:2])
def test_scores_that_repeat_are_sorted_instead_of_walked(size, layer):
    """Many equal scores: their segments are not walked entry by entry (4.3 to 5 times as long), and the list is sorted without
    a selection."""
    plain, ties = _topk_us(*size, layer=layer), _topk_us(*size, distinct=64, layer=layer)
    print(f"[time] {'layer' if layer else 'select'} {size}: independent {plain:.1f} us, 64 different keys {ties:.1f} us", flush=True)
    assert ties < 3.5 * plain

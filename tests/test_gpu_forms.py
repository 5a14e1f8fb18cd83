"""The two forms of the Group-GEMM launch (planned tiles, and the narrow items
that launches with few tiles are cut into) against the oracle, at the edges of
their tiles: rows around 16 / 32 / 64 / 128, channels around the item widths
(64, 128) and the tile widths (256, 512), reductions with and without slices
(of at least 8 k blocks in a narrow linear, 12 in a narrow block); which form a
launch takes; and the launches in front, routing and the encoding of long
inputs."""

import numpy as np
import pytest

from oracle import mxmoe_oracle as O
from paper_2505_05799_amd import mxmoe as M
from paper_2505_05799_amd import workloads as W
from tests.gpuhelp import say, torch_mod, upload_inputs
from tests.stagewise import check_forward
from tests.test_gpu_forward import run_block
from tests.test_gpu_kernels import _check_linear, _linear_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", W.ALL_SCHEMES, ids=lambda s: s.name)
@pytest.mark.parametrize("m,n,k", [(1, 528, 1536), (16, 144, 640), (17, 1040, 512), (33, 656, 1536),
                                   (64, 272, 384), (97, 400, 1536), (129, 784, 256)])
def test_narrow_linear(scheme, m, n, k):
    """At most 512 tiles: the narrow form (the rows' halves and the channels'
    quarters past the edges hold no work)."""
    for act in ("bf16", "fp16"):
        q, a, got, _ = _linear_case(scheme, act, m, n, k, m + n + k)
        _check_linear(q, a, got, act)


@pytest.mark.parametrize("scheme", W.ALL_SCHEMES, ids=lambda s: s.name)
@pytest.mark.parametrize("m,n", [(16, 528), (33, 656), (97, 528), (129, 656)])
def test_narrow_linear_slices(scheme, m, n):
    """Slices of several channel items, the last one ragged."""
    for act in ("bf16", "fp16"):
        q, a, got, split = _linear_case(scheme, act, m, n, 4096, m + n)
        assert split >= 2
        _check_linear(q, a, got, act)


@pytest.mark.parametrize("act,T", [("bf16", 9), ("fp16", 70)])
def test_narrow_block_slices(act, T):
    """Both launches narrow and several of their groups sliced: the plan's
    records against the oracle's with 12 k blocks a slice (and a partial buffer
    that refuses no slice), each group with areas and counters of its own, and
    the block against the oracle."""
    from tests.test_gpu_configs import PF_N, plan_misc
    torch = torch_mod()
    sch = [(W.W4G128, W.W4G128, W.W3G128), (W.W8A8, W.W8A8, W.FP8), (W.W3G128, W.W3G128, W.W4A4G128)]
    blk = W.random_small_block(77 + T, T=T, H=3072, F=3072, E=2, k=1, n_shared=1, F_shared=3200, act=act, schemes=sch)
    mb, y = run_block(blk)
    lay = mb.workspace_layout(T)
    misc = plan_misc(mb, T, 3, lay["plan_queue_cap"])
    assert misc[9] == 4
    rec = mb.ws_view("plan", torch.int32, 2 * 3 * PF_N, T).cpu().numpy().reshape(2, 3, PF_N)
    ms = [int((blk.topk_ids == e).sum()) for e in range(2)] + [T]
    for ph in (0, 1):
        lins = [blk.linears[g][0 if ph == 0 else 2] for g in range(3)]
        want, _ = O.tile_plan(ms, lins, ph, M.get_tile_costs(), partial_floats=1 << 40, nwg=int(misc[8]), min_kb=12)
        assert sum(w["split"] > 1 for w in want) >= 2
        for g, w in enumerate(want):
            got = dict(zip(("m", "cfg", "mtiles", "ntiles", "cost", "rank", "split", "pbase", "cbase"),
                           rec[ph, g][[1, 2, 3, 4, 6, 7, 8, 9, 10]].tolist()))
            assert got == {"m": ms[g], **{f: w[f] for f in got if f != "m"}}, (ph, g)
    say(f"T={T} {act}: {check_forward(mb, blk, y).line()}")


@pytest.mark.parametrize("scheme", W.ALL_SCHEMES, ids=lambda s: s.name)
@pytest.mark.parametrize("m", [4133, 7201])
def test_wide_linear(scheme, m):
    """(1 + m / 64) tile rows of 9 (m = 4133) or 5 channel tiles are more than
    512 tiles of few weight bytes each: the planned tiles themselves."""
    n = 2064 if m == 4133 else 1040
    for act in ("bf16", "fp16"):
        q, a, got, _ = _linear_case(scheme, act, m, n, 384, m + n)
        _check_linear(q, a, got, act)


BLOCKS = [
    [(W.W4G128,) * 3, (W.W8A8, W.W8A8, W.W2G128), (W.W4A4,) * 3, (W.W16, W.W16, W.W3G128), (W.W3G128,) * 3,
     (W.W8G128, W.W8G128, W.W4A4), (W.W2G128, W.W2G128, W.W8A8)],
    [(W.MXFP4,) * 3, (W.FP8,) * 3, (W.W4A4G128,) * 3, (W.W4A4F6, W.W4A4F6, W.W4G128), (W.FP8, W.FP8, W.MXFP4),
     (W.W4A4G128, W.W4A4G128, W.W4A4F6), (W.W4G128, W.W4G128, W.FP8)],
]


@pytest.mark.parametrize("act", ["bf16", "fp16"])
@pytest.mark.parametrize("mix", [0, 1])
@pytest.mark.parametrize("T", [41, 3000])   # narrow; 594 and more gate|up tiles: wide
def test_block_forms(T, mix, act):
    blk = W.random_small_block(31 + T, T=T, H=256, F=768, E=6, k=2, n_shared=1, F_shared=384, act=act,
                               schemes=BLOCKS[mix], skew=1.0)
    mb, y = run_block(blk)
    rep = check_forward(mb, blk, y)
    say(f"T={T} mix {mix} {act}: {rep.line()}")


@pytest.mark.parametrize("E,k,T", [(60, 4, 1), (60, 4, 1024), (61, 8, 129), (70, 4, 40), (60, 9, 40), (252, 3, 50), (260, 3, 50)])
def test_routing_forms(E, k, T):
    """Routing inside the plan launch (at most 4096 pairs and 256 groups), with
    the router (at most 64 experts, k <= 8) and without, and in launches of its
    own: from logits and from the ids and weights they give, the same bits; the
    routing arrays and the block against the oracle."""
    torch = torch_mod()
    blk = W.random_small_block(5 + E + k, T=T, H=128, F=128, E=E, k=k, n_shared=1, F_shared=128, act="bf16",
                               schemes=[(s,) * 3 for s in (W.W8A8, W.W4A4, W.W4G128, W.FP8)] * (E // 4) +
                               [(W.W8A8,) * 3] * (E % 4 + 1))
    logits, _ = W.router_logits(T, E, seed=E, zipf_s=1.0)
    blk.topk_ids, blk.topk_w = O.router_topk(logits, k)
    blk.topk_ids = np.ascontiguousarray(blk.topk_ids, dtype=np.int32)
    mb = M.MoEBlock(blk)
    x, ids, _ = upload_inputs(blk)
    lg = torch.from_numpy(logits).cuda()
    gids, gw, _ = M.router_topk(lg, k)
    assert torch.equal(gids, ids)
    y1 = mb.forward(x, None, None, router_logits=lg).clone()
    y2 = mb.forward(x, gids, gw)
    torch.cuda.synchronize()
    assert torch.equal(y1.view(torch.int16), y2.view(torch.int16))
    r = O.route(blk.topk_ids, E)
    for f, n in (("counts", E), ("offsets", E + 1), ("sorted_pair", T * k), ("inv", T * k)):
        assert np.array_equal(mb.ws_view(f, torch.int32, n, T).cpu().numpy(), r[f]), f
    blk.topk_w = gw.cpu().numpy()
    say(f"E={E} k={k} T={T}: {check_forward(mb, blk, y2).line()}")


QUANT_ACT = [s for s in W.ALL_SCHEMES if s.a_bits < 16]


@pytest.mark.parametrize("scheme", QUANT_ACT, ids=lambda s: s.name)
@pytest.mark.parametrize("m,n,k", [(8, 48, 4224), (9, 48, 4224), (9, 16, 6144), (8, 16, 6144), (8, 48, 12288),
                                   (41, 16, 8192), (1537, 16, 6144), (3, 16, 16512), (2, 16, 32896)])
def test_linear_long_rows(scheme, m, n, k):
    """Inputs of more than 4096 columns, on both sides of the lines where their
    encoding moves from the plan launch to one of its own, and of more columns
    than a workgroup holds in registers."""
    for act in ("bf16", "fp16"):
        q, a, got, _ = _linear_case(scheme, act, m, n, k, m + n + k)
        _check_linear(q, a, got, act)


@pytest.mark.parametrize("scheme", QUANT_ACT, ids=lambda s: s.name)
def test_long_rows_are_read_in_few_round_trips(scheme):
    """16 rows of 28672 columns against 14336: the weights of the second half
    (up to 29 MB) stream in about 10 us.  A wavefront that reads its row in
    1 KB round trips, twice, adds 56 of them, 28 us and more."""
    torch = torch_mod()

    def us(k):
        q = W.QLinear(scheme, 2048, k, *_random_operands(scheme, 2048, k))
        pl = M.PackedLinear(q, "bf16")
        a = torch.randn(16, k, device="cuda").bfloat16()
        for _ in range(3):
            M.linear_forward(pl, a)
        best = 1e9
        for _ in range(8):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(20):
                M.linear_forward(pl, a)
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1) * 1e3 / 20)
        return best

    short, long = us(14336), us(28672)
    say(f"{scheme.name}: 16 x 14336 {short:.1f} us, 16 x 28672 {long:.1f} us")
    assert long - short < 20.0


def _random_operands(s, n, k):
    """Codes and scales of a quantized scheme's formats (their values do not matter)."""
    rng = np.random.default_rng(k)
    if s.fmt == 1:
        return rng.integers(0, 16, (n, k), dtype=np.uint8), np.full((n, k // 32), 127, np.uint8)
    if s.fmt == 2:
        return rng.integers(0, 0x70, (n, k), dtype=np.uint8), np.full(n, 0.01, np.float32)
    top = (1 << (s.w_bits - 1)) - 1
    codes = rng.integers(-top, top + 1, (n, k), dtype=np.int8)
    if s.w_group > 0:
        return codes, np.full((n, k // s.w_group), 0.01, np.float16)
    return codes, np.full(n, 0.01, np.float32)


def _linear_items(s, m, n, k):
    """Items a tile of the linear's launch is claimed in (the plan's misc[9])."""
    torch = torch_mod()
    pl = M.PackedLinear(W.QLinear(s, n, k, *_random_operands(s, n, k)), "bf16")
    _, ws = M.linear_forward(pl, torch.zeros(m, k, dtype=torch.bfloat16, device="cuda"), return_ws=True)
    torch.cuda.synchronize()
    cap = (m // 1024 + 3) * (n // 512 + 2) // 8 + 2 + 16384 // 8 + 1     # plan_queue_cap
    at = 28 + 2 * 8 * cap * 3 + 2 * 8 * 4 + 9                            # records, order, entries, counters
    return int(ws[4 * at: 4 * at + 4].view(torch.int32).item())


@pytest.mark.parametrize("scheme,m,n,k,items", [
    (W.W4A4, 31, 1040, 512, 4), (W.FP8, 1984, 4096, 256, 1), (W.MXFP4, 2021, 3408, 256, 1),
    (W.FP8, 500, 8192, 128, 1), (W.FP8, 500, 7936, 128, 4), (W.W8A8, 1984, 4096, 256, 4),
    (W.W8A8, 100, 81920, 1536, 1), (W.W8A8, 100, 81664, 1536, 4),
    (W.W4A4G128, 6400, 1024, 256, 1), (W.W4A4G128, 6300, 1024, 256, 4),
    (W.W4A4F6, 512, 4096, 12288, 4), (W.W8A8, 512, 4096, 12288, 1), (W.W8A8, 512, 4096, 12160, 4), (W.W8A8, 300, 4096, 12288, 4)],
    ids=lambda v: getattr(v, "name", str(v)))
def test_linear_form(scheme, m, n, k, items):
    """Launches of few tiles are narrow (items 4); those whose tiles fill the
    chip are not: 320 to 512 (256 of FP8 and MXFP4, 400 of w4a4-g128), or 60 to
    64 of 8- or 16-bit weights and at least 96 k blocks."""
    assert _linear_items(scheme, m, n, k) == items


@pytest.mark.parametrize("E,T,items", [(8, 2048, 4), (8, 2300, 1), (10, 2550, 4), (10, 2560, 1)])
def test_block_form(E, T, items):
    """Experts of 4 channel tiles of FP8, which leave the narrow form at 512 rows
    each, 256 tiles and ten super-tiles (a ninth row tile begins another)."""
    from tests.test_gpu_configs import plan_misc
    blk = W.random_small_block(T, T=T, H=256, F=512, E=E, k=2, act="bf16", schemes=[(W.FP8,) * 3] * E)
    mb, y = run_block(blk)
    assert plan_misc(mb, T, E, mb.workspace_layout(T)["plan_queue_cap"])[9] == items
    say(f"E={E} T={T}: {check_forward(mb, blk, y).line()}")

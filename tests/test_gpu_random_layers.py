"""Seeded random layers: lengths, head sizes, mode mixes, band widths, offsets,
column sets, batch, text prefix and dense split drawn at random; bf16 and FP8
paths against their oracles on all rows."""
import numpy as np
import pytest
import torch

from paper_2506_03065_amd import binding as svd
from paper_2506_03065_amd import workloads as W
from parity_util import check_layer, run_planned
from test_gpu_fp8 import check_layer_fp8, run_fp8

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run_plan(wl, q, k, v, **options):
    desc = svd.desc_of(q)
    ws = torch.empty(svd.svd_plan_workspace_bytes(desc, wl.strategy_table, wl.pattern_params, **options), dtype=torch.uint8, device=DEV)
    plan = svd.svd_plan_create(desc, wl.strategy_table, wl.pattern_params, workspace=ws, **options)
    out = torch.full_like(q, float("nan"))
    svd.svd_attn_forward_planned(plan, q, k, v, out)
    torch.cuda.synchronize()
    return out, plan, ws


def random_layer(seed):
    rng = np.random.default_rng(1000 + seed)
    D = int(rng.choice([64, 128]))
    L = int(rng.integers(260, 2200))
    H = int(rng.integers(3, 9))
    B = int(rng.choice([1, 1, 2]))
    text = int(rng.choice([0, 0, 256])) if L > 600 else 0
    table = rng.integers(0, 5, H).astype(np.int32)
    table[rng.integers(0, H)] = W.MULTIDIAG          # at least one of the harder modes
    params = []
    for m in table:
        p = {"half_width": 0, "offsets": (), "cols": ()}
        if m == W.DIAG:
            p["half_width"] = int(rng.integers(0, L // 2))
            p["offsets"] = (0,)
        elif m == W.MULTIDIAG:
            step = int(rng.integers(20, max(21, L // 3)))
            ks = rng.choice(np.arange(-4, 5), size=int(rng.integers(1, 6)), replace=False)
            offs = sorted({0} | {int(k) * step for k in ks})      # offset 0 keeps every row non-empty
            p["half_width"] = int(rng.integers(0, max(1, step // 2)))
            p["offsets"] = tuple(offs)
        elif m == W.VSTRIPE:
            n = int(rng.integers(1, max(2, L // 4)))
            p["cols"] = tuple(int(c) for c in np.sort(rng.choice(L, size=n, replace=False)))
        if text and m >= W.DIAG:
            p["text_tokens"] = text
        params.append(p)
    split = int(rng.choice([0, 0, 1, 2, 5]))
    wl = W.Workload(f"random{seed}", -1, B, H, L, D, max(8, L // 5), 5, text, table, params, 4000 + seed)
    return wl, split


@pytest.mark.parametrize("seed", list(range(12)) + [23, 45])   # the last two: narrow-band heads with the largest single-element deviations seen
def test_random_layer(seed):
    wl, split = random_layer(seed)
    q, k, v = (t.to(DEV) for t in W.make_qkv(wl))
    out = run_planned(wl, q, k, v, dense_split=split)
    check_layer(wl, q, k, v, out)
    out8, _ = run_fp8(wl, q, k, v, dense_split=split)
    check_layer_fp8(wl, q, k, v, out8)
    for h in range(wl.H):
        if wl.strategy_table[h] == W.SKIP:
            assert not out[:, h].view(torch.int16).any() and not out8[:, h].view(torch.int16).any()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("step,w", [(17, 3), (9, 2), (33, 0), (64, 31), (5, 2)])
def test_several_runs_in_one_tile(D, step, w):
    """Seven bands `step` apart: a key tile is crossed by up to seven runs (step 5 merges all into one), with their edges
    in every place of a lane's elements and past both ends of the sequence, in bf16 and FP8."""
    L = 777
    params = {"half_width": w, "offsets": tuple(i * step for i in range(-3, 4))}
    wl = W.Workload("runs", -1, 1, 2, L, D, 111, 7, 0, np.full(2, W.MULTIDIAG, dtype=np.int32), [params, dict(params)], 97)
    q, k, v = (t.to(DEV) for t in W.make_qkv(wl))
    check_layer(wl, q, k, v, run_planned(wl, q, k, v))
    out8, _ = run_fp8(wl, q, k, v)
    check_layer_fp8(wl, q, k, v, out8)


FORMS = {"table": {}, "layer": {"single_launch": 1}, "groups": {"single_launch": 2}, "groups-large": {"single_launch": 2, "block_q": 256}}


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("step,w", [(17, 3), (9, 2), (33, 0), (64, 31), (5, 2)])
def test_several_runs_in_one_tile_in_every_launch_form(D, step, w, form):
    """Seven bands `step` apart: a key tile is crossed by up to seven runs (step 5 merges all into one), with their edges
    in every place of a lane's elements and past both ends of the sequence, and a band over positions in any frames; in bf16
    from the table (four waves), the layer kernel and a launch per group on either query tile, and in FP8 from the table and
    per group."""
    L = 777
    params = {"half_width": w, "offsets": tuple(i * step for i in range(-3, 4))}
    window = {"half_width": step * 7 + 6, "rearranged": (0, 111, 7)}
    wl = W.Workload("runs", -1, 1, 3, L, D, 111, 7, 0, np.full(3, W.MULTIDIAG, dtype=np.int32), [params, dict(params), window], 97)
    q, k, v = (t.to(DEV) for t in W.make_qkv(wl))
    options = dict(FORMS[form])
    if "block_q" in options:
        options["block_k"] = 64 if D == 128 else 128
    out, plan, _ = run_plan(wl, q, k, v, **options)
    table, single = plan.table()["bf16"], plan.single_launch()
    sizes = {g["block_q"] for g in plan.groups()}
    plan.close()
    assert (table, single) == {"table": (4, False), "layer": (0, True)}.get(form, (0, False))
    assert form != "groups-large" or sizes == {256}
    check_layer(wl, q, k, v, out)
    if form in ("table", "groups"):
        out8, _ = run_fp8(wl, q, k, v, dense_split=0 if form == "table" else 1)
        check_layer_fp8(wl, q, k, v, out8)

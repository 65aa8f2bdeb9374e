"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import sparse_attention as O
from paper_2506_03065_amd import binding as svd
from paper_2506_03065_amd import workloads as W
from parity_util import assert_close, check_layer, f64, run_planned

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _cuda(ts):
    return [t.to(DEV) for t in ts]


def test_tiny_all_rows():
    wl = W.tiny()
    q, k, v = _cuda(W.make_qkv(wl))
    out = run_planned(wl, q, k, v)
    check_layer(wl, q, k, v, out)


@pytest.mark.parametrize("L,D,H,seed,B", [(333, 64, 5, 7, 1), (200, 128, 5, 11, 1), (1000, 64, 5, 3, 1),
                                           (1000, 128, 5, 4, 1), (77, 128, 4, 5, 1), (31, 64, 4, 6, 1),
                                           (520, 128, 10, 8, 2), (700, 64, 5, 9, 2),
                                           (1, 64, 5, 12, 1), (2, 128, 5, 13, 2), (16, 64, 5, 14, 1)])
def test_small_ragged_all_rows(L, D, H, seed, B):
    wl = W.small(L=L, D=D, H=H, seed=seed, B=B)
    q, k, v = _cuda(W.make_qkv(wl))
    out = run_planned(wl, q, k, v)
    check_layer(wl, q, k, v, out)
    skipped = [h for h in range(wl.H) if wl.strategy_table[h] == W.SKIP]
    for h in skipped:
        assert not out[:, h].view(torch.int16).any(), "skipped head must be exact zeros"


@pytest.mark.parametrize("D", [64, 128])
def test_dense_entry_point(D):
    wl = W.small(L=777, D=D, H=3, seed=21)
    wl.strategy_table[:] = W.DENSE
    q, k, v = _cuda(W.make_qkv(wl))
    out = torch.full_like(q, float("nan"))
    svd.svd_dense_attn_forward(q, k, v, out)
    torch.cuda.synchronize()
    check_layer(wl, q, k, v, out)


def test_one_shot_entry_point_and_plan_reuse():
    wl = W.small(L=600, D=128, H=5, seed=31)
    q, k, v = _cuda(W.make_qkv(wl))
    nbytes = svd.svd_plan_workspace_bytes(svd.desc_of(q), wl.strategy_table, wl.pattern_params)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    out = torch.full_like(q, float("nan"))
    for _ in range(2):   # second call reuses the compiled plan
        out.fill_(float("nan"))
        svd.sparse_vdit_attn_forward(q, k, v, wl.strategy_table, wl.pattern_params, out, ws)
        torch.cuda.synchronize()
        check_layer(wl, q, k, v, out)
    # a different table through the same workspace recompiles
    wl2 = W.small(L=600, D=128, H=5, seed=32)
    wl2.strategy_table = wl.strategy_table[::-1].copy()
    wl2.pattern_params = wl.pattern_params[::-1]
    svd.sparse_vdit_attn_forward(q, k, v, wl2.strategy_table, wl2.pattern_params, out, ws)
    torch.cuda.synchronize()
    check_layer(wl2, q, k, v, out)


def test_strided_token_major_layout():
    """[B, L, H, D] storage viewed as [B, H, L, D] (the merged-head layout)."""
    wl = W.small(L=450, D=64, H=5, seed=41)
    q, k, v = _cuda(W.make_qkv(wl))
    qs, ks, vs = (t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for t in (q, k, v))
    assert not qs.is_contiguous()
    out = torch.full_like(qs, float("nan"))
    assert out.stride() == qs.stride()
    run_planned(wl, qs, ks, vs, out)
    check_layer(wl, q, k, v, out)


def test_wide_patterns_equal_dense_and_edge_parameters():
    L, D = 500, 64
    table = np.asarray([W.DENSE, W.DIAG, W.MULTIDIAG, W.VSTRIPE, W.DIAG, W.MULTIDIAG, W.VSTRIPE], dtype=np.int32)
    params = [{}, {"half_width": L - 1}, {"half_width": 60, "offsets": tuple(range(-480, 481, 120))},
              {"cols": tuple(range(L))}, {"half_width": 0}, {"half_width": 1, "offsets": (0, 3, 7, 200, -200)},
              {"cols": (499,)}]
    wl = W.Workload("edges", -1, 1, len(table), L, D, 100, 5, 0, table, params, 51)
    q, k, v = W.make_qkv(wl)
    for t in (q, k, v):          # same inputs for the heads compared with the dense one
        t[:, 1:4] = t[:, 0:1]
    q, k, v = _cuda((q, k, v))
    out = run_planned(wl, q, k, v)
    check_layer(wl, q, k, v, out)
    for h in (1, 2, 3):
        assert_close(f64(out[0, h]), f64(out[0, 0]), f"full-width head {h} vs dense")


def test_closed_forms_constant_v_and_zero_q():
    wl = W.small(L=900, D=128, H=5, seed=61)
    q, k, v = _cuda(W.make_qkv(wl))
    vc = torch.full_like(v, 0.625)
    out = run_planned(wl, q, k, vc)
    for h in range(wl.H):
        want = 0.0 if wl.strategy_table[h] == W.SKIP else 0.625
        assert torch.allclose(out[0, h].float(), torch.full_like(out[0, h].float(), want), atol=4e-3)
    out = run_planned(wl, torch.zeros_like(q), k, v)
    vf = f64(v[0])
    for h in range(wl.H):
        mode, p = int(wl.strategy_table[h]), wl.pattern_params[h]
        if mode == W.SKIP:
            continue
        prefix = np.concatenate([np.zeros((1, wl.D)), np.cumsum(vf[h], axis=0)])
        want = np.zeros((wl.L, wl.D))
        if mode == W.DENSE:
            want[:] = vf[h].mean(axis=0)
        elif mode == W.VSTRIPE:
            want[:] = vf[h][list(p["cols"])].mean(axis=0)
        else:
            w = p["half_width"]
            for i in range(wl.L):
                tot, cnt = 0.0, 0
                for o in p["offsets"]:
                    lo, hi = max(0, i + o - w), min(wl.L, i + o + w + 1)
                    if hi > lo:
                        tot, cnt = tot + prefix[hi] - prefix[lo], cnt + hi - lo
                want[i] = tot / cnt
        assert_close(f64(out[0, h]), want, f"zero-q mean, head {h}")


def test_errors_leave_output_untouched():
    wl = W.small(L=300, D=64, H=5, seed=71)
    q, k, v = _cuda(W.make_qkv(wl))
    out = torch.full_like(q, 3.0)
    ws = torch.empty(1 << 16, dtype=torch.uint8, device=DEV)
    bad = wl.strategy_table.copy()
    bad[0] = 9
    with pytest.raises(svd.SvdError) as e:
        svd.sparse_vdit_attn_forward(q, k, v, bad, wl.pattern_params, out, ws)
    assert e.value.status == 5
    with pytest.raises(svd.SvdError) as e:
        svd.sparse_vdit_attn_forward(q, k, v, wl.strategy_table, wl.pattern_params, out, ws[:16])
    assert e.value.status == 8
    with pytest.raises(svd.SvdError) as e:   # misaligned base pointer
        svd.svd_dense_attn_forward(q.view(-1)[4:4 + 64 * 64].view(1, 1, 64, 64), k, v, out)
    assert e.value.status == 4
    torch.cuda.synchronize()
    assert (out == 3.0).all()
    # a plan compiled for another block shape can be inspected but not launched
    desc = svd.desc_of(q)
    plan = svd.svd_plan_create(desc, wl.strategy_table, wl.pattern_params, 32, 32, workspace=ws)
    with pytest.raises(svd.SvdError) as e:
        svd.svd_attn_forward_planned(plan, q, k, v, out)
    assert e.value.status == 9
    assert (out == 3.0).all()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("profile", ["rising", "falling", "late_outlier", "very_negative"])
def test_peaked_scores_move_the_softmax_reference(D, profile):
    """Score profiles along the key axis that make the running reference of the
    online softmax move many times (rising), never after the first tile
    (falling), once by a large jump near the end (late_outlier), or that sit
    far below zero everywhere (very_negative: an unset reference must not be
    taken for zero).  Logits reach 50 to 180 in magnitude, far beyond what
    N(0,1) inputs give."""
    L, H = 1500, 5
    wl = W.small(L=L, D=D, H=H, seed=41)
    q, k, v = W.make_qkv(wl)
    j = torch.arange(L, dtype=torch.float32)
    if profile == "rising":
        gain = 0.25 + 2.75 * j / L
    elif profile == "falling":
        gain = 3.0 - 2.75 * j / L
    elif profile == "late_outlier":
        gain = torch.ones(L)
        gain[L - 37] = 5.0
    else:
        gain = torch.full((L,), 8.0)
    # every query looks along +u; key j looks along gain[j] * u (minus for very_negative)
    u = torch.nn.functional.normalize(torch.ones(D), dim=0) * (D ** 0.5)
    sign = -1.0 if profile == "very_negative" else 1.0
    q = (0.3 * q.float() + 2.0 * u).to(torch.bfloat16)
    k = (0.3 * k.float() + sign * gain[None, None, :, None] * u).to(torch.bfloat16)
    q, k, v = _cuda([q, k, v])
    out = run_planned(wl, q, k, v)
    check_layer(wl, q, k, v, out)


def band_edges_layer(L, D, w):
    far = L - 1 - w // 2
    params = [{"half_width": w}, {"half_width": w, "offsets": (-3 * w - 40, 0, 3 * w + 40)},
              {"half_width": max(w, far // 2), "offsets": (far // 2, 0)}, {"half_width": max(w, far // 2), "offsets": (0, -far // 2)}]
    wl = W.small(L=L, D=D, H=4, seed=53)
    wl.strategy_table = np.asarray([W.DIAG, W.MULTIDIAG, W.MULTIDIAG, W.MULTIDIAG], dtype=np.int32)
    wl.pattern_params = [dict(p, offsets=p.get("offsets", ()), cols=()) for p in params]
    return wl


@pytest.mark.parametrize("L,D", [(449, 64), (449, 128), (640, 128)])
@pytest.mark.parametrize("w", [0, 1, 15, 16, 31, 32, 33, 64, 100, 127, 128, 130])
def test_band_edges_in_every_place_of_a_block(L, D, w):
    """Bands whose edges cross the 32 x 32 blocks of a tile one at a time, both in one block (2 w + 1 < 32), on a
    block's border, and together with the end of the sequence: one diagonal head, one with several bands, and the
    same band shifted off the diagonal so that only its lower or only its upper edge lies inside the sequence."""
    wl = band_edges_layer(L, D, w)
    q, k, v = _cuda(W.make_qkv(wl))
    check_layer(wl, q, k, v, run_planned(wl, q, k, v))


@pytest.mark.parametrize("layout", ["bhld", "blhd"])
@pytest.mark.parametrize("L,D", [(1, 64), (77, 128), (449, 64), (449, 128), (1000, 64), (1001, 128), (1930, 64)])
@pytest.mark.parametrize("options", [{}, {"single_launch": 2}, {"single_launch": 2, "dense_split": 3}, {"single_launch": 1}],
                         ids=["table", "groups", "split", "layer"])
def test_rows_behind_the_last_one_are_not_read(layout, L, D, options):
    """Q, K, V and O as views of larger storage in which every row behind a head's last one holds NaN: a key row past the
    end is no row of the tensor for the loads of a ragged last tile either (a masked probability of 0 times NaN is NaN)."""
    wl = W.small(L=L, D=D, H=5, seed=57, B=2)
    pad = 192
    views = []
    for t in W.make_qkv(wl) + [torch.full((wl.B, wl.H, L, D), float("nan"), dtype=torch.bfloat16)]:
        store = torch.full((wl.B, wl.H, L + pad, D) if layout == "bhld" else (wl.B, L + pad, wl.H, D), float("nan"),
                           dtype=torch.bfloat16, device=DEV)
        view = store[:, :, :L] if layout == "bhld" else store[:, :L].permute(0, 2, 1, 3)
        view.copy_(t)
        views.append((store, view))
    (_, q), (_, k), (_, v), (out_store, out) = views
    desc = svd.desc_of(q)
    ws = torch.empty(svd.svd_plan_workspace_bytes(desc, wl.strategy_table, wl.pattern_params, **options), dtype=torch.uint8, device=DEV)
    plan = svd.svd_plan_create(desc, wl.strategy_table, wl.pattern_params, workspace=ws, **options)
    svd.svd_attn_forward_planned(plan, q, k, v, out)
    torch.cuda.synchronize()
    plan.close()
    check_layer(wl, q, k, v, out)
    behind = out_store[:, :, L:] if layout == "bhld" else out_store[:, L:]
    assert torch.isnan(behind).all(), "a row behind the last one was written"


@pytest.mark.parametrize("D,options", [(64, {}), (128, {}), (128, {"single_launch": 1})])
def test_rows_behind_the_last_one_past_32_bits(D, options):
    """The largest row stride: the last row starts below byte 2^32 of its head, the rows that fill its key tile lie past
    it.  All storage between and behind the rows (mapped, and as far as those rows reach) holds NaN."""
    L, rows_of_tiles, H = 1985, 2048, 3
    stride = (2 ** 32 - 1) // L // 16 * 8
    assert L * stride * 2 < 2 ** 32 < (rows_of_tiles - 1) * stride * 2
    wl = W.small(L=L, D=D, H=H, seed=58)   # dense, diagonal, multi-diagonal
    store = torch.full((rows_of_tiles * stride + 16 * 128,), float("nan"), dtype=torch.bfloat16, device=DEV)
    q, k, v, out = (torch.as_strided(store, (1, H, L, D), (H * 128, 128, stride, 1), i * H * 128) for i in range(4))
    for view, t in zip((q, k, v), W.make_qkv(wl)):
        view.copy_(t)
    desc = svd.desc_of(q)
    ws = torch.empty(svd.svd_plan_workspace_bytes(desc, wl.strategy_table, wl.pattern_params, **options), dtype=torch.uint8, device=DEV)
    plan = svd.svd_plan_create(desc, wl.strategy_table, wl.pattern_params, workspace=ws, **options)
    svd.svd_attn_forward_planned(plan, q, k, v, out)
    torch.cuda.synchronize()
    plan.close()
    check_layer(wl, q, k, v, out, rows=np.asarray([0, 1, 127, 128, 993, 1856, 1919, 1920, 1983, 1984]))
    del store


@pytest.mark.parametrize("L,stride,D", [(9256395, 232, 128), (10737418, 200, 128), (16777215, 128, 64)])
def test_padding_of_a_column_list_when_the_head_ends_close_to_32_bits(L, stride, D):
    """Two heads whose last row ends within 256 bytes of byte 2^32, and the longest of contiguous rows at D = 64: the padding of
    a column list must not reach into that row, whose V is not finite here."""
    assert D == 64 or 2 ** 32 - 256 < (L - 1) * stride * 2 + D * 2 < 2 ** 32
    cols = np.unique(np.random.default_rng(7).integers(0, L - 1, 70)).astype(np.int32)
    table, params = np.asarray([W.VSTRIPE], dtype=np.int32), [{"cols": cols}]
    q, v, out = (torch.as_strided(torch.empty(L * stride, dtype=torch.bfloat16, device=DEV), (1, 1, L, D), (L * stride, L * stride, stride, 1))
                 for _ in range(3))
    gen = torch.Generator(device=DEV).manual_seed(59)
    for t in (q, v):
        t.normal_(generator=gen)
    v[:, :, L - 1] = float("inf")
    out.fill_(float("nan"))
    desc = svd.desc_of(q)
    ws = torch.empty(svd.svd_plan_workspace_bytes(desc, table, params), dtype=torch.uint8, device=DEV)
    plan = svd.svd_plan_create(desc, table, params, workspace=ws)
    assert plan.table()["bf16"] == 4   # columns are read through their list
    svd.svd_attn_forward_planned(plan, q, q, v, out)
    torch.cuda.synchronize()
    plan.close()
    rows, idx = [0, 1, 127, 128, L // 2, L - 2, L - 1], torch.as_tensor(cols.astype(np.int64), device=DEV)
    assert torch.isfinite(out[0, 0, :: 4099]).all() and torch.isfinite(out[0, 0, -300:]).all()
    s = q[0, 0, rows].double() @ q[0, 0, idx].double().T / D ** 0.5
    want = torch.softmax(s, 1) @ v[0, 0, idx].double()
    for i, r in enumerate(rows):
        assert_close(f64(out[0, 0, r: r + 1]), f64(want[i: i + 1]), f"row {r}")


@pytest.mark.parametrize("L,D,split", [(1000, 64, 2), (1000, 64, 3), (1000, 128, 5), (777, 128, 8), (130, 64, 8),
                                       (60, 128, 4)])
def test_dense_key_range_split(L, D, split):
    """Dense heads computed in `split` key-range chunks and merged (forced through
    the plan option; chunk counts above the number of key tiles are capped)."""
    wl = W.small(L=L, D=D, H=5, seed=51, B=2)
    q, k, v = _cuda(W.make_qkv(wl))
    desc = svd.desc_of(q)
    plan = svd.svd_plan_create(desc, wl.strategy_table, wl.pattern_params, dense_split=split,
                               workspace=torch.empty(svd.svd_plan_workspace_bytes(
                                   desc, wl.strategy_table, wl.pattern_params, dense_split=split),
                                   dtype=torch.uint8, device=DEV))
    n_key_tiles = -(-L // svd.svd_default_blocks(D)[1])
    assert plan.dense_split() == min(split, n_key_tiles)
    plan.close()
    out = run_planned(wl, q, k, v, dense_split=split)
    check_layer(wl, q, k, v, out)


def test_dense_split_with_peaked_scores():
    """Chunks whose reference exponents differ by hundreds must merge exactly."""
    L, D = 1500, 64
    wl = W.small(L=L, D=D, H=5, seed=52)
    q, k, v = W.make_qkv(wl)
    gain = 0.25 + 2.75 * torch.arange(L, dtype=torch.float32) / L
    u = torch.ones(D)
    q = (0.3 * q.float() + 2.0 * u).to(torch.bfloat16)
    k = (0.3 * k.float() + gain[None, None, :, None] * u).to(torch.bfloat16)
    q, k, v = _cuda([q, k, v])
    out = run_planned(wl, q, k, v, dense_split=4)
    check_layer(wl, q, k, v, out)

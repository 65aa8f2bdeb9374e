"""The whole layer from a table of items: the table on the host model of the launches (every output row
stored once, every word inside the workspace, the chunks of cut items complete), and items of every kind
cut into chunks on the GPU against the oracle."""
import os
import subprocess

import numpy as np
import pytest
import torch

from paper_2506_03065_amd import binding as svd
from paper_2506_03065_amd import workloads as W
from parity_util import check_layer, run_planned
from test_gpu_fp8 import check_layer_fp8, run_fp8
from test_gpu_random_layers import random_layer
from test_host_launch_model import CSRC, ROOT, STUB, layer_text, replay, run  # noqa: F401  (replay: the fixture)


@pytest.mark.parametrize("cu", [8, 256])
def test_random_layers_from_the_table(replay, tmp_path, cu):
    layers = [layer_text(random_layer(seed)[0], 0, rounds=1, cu=cu) for seed in range(16)]
    wl = W.small(L=900, D=128, H=6, seed=17)
    wl.pattern_params[2] = {"half_width": 2 * 5 + 4, "rearranged": (0, 180, 5)}
    layers.append(layer_text(wl, 0, rounds=1, cu=cu))
    layers += [layer_text(W.small(L=L, D=D, H=5, seed=3), 0, rounds=1, cu=cu) for L in (1, 127, 128, 129, 257) for D in (64, 128)]
    res = run(replay, tmp_path, layers)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]


def tables_of(res):
    """{(waves, cut items)} of the bf16 tables that the harness walked."""
    words = [line.split() for line in res.stdout.splitlines() if line.startswith("grid:")]
    return {(int(w[2]), int(w[6]) > 0) for w in words if w[8] == "0"}


def large_tile_layer(L, n_dense, diag_w, B=1):
    """D = 64 with enough key tiles for eight-wave work-groups: dense heads, a wide band (a group on the 256-row tile), a
    narrow multi-diagonal band (a group on the 128-row tile, whose lists on the large one are appended for the table), a
    stripe head, a skipped one."""
    table = np.asarray([W.DENSE] * n_dense + [W.DIAG, W.MULTIDIAG, W.VSTRIPE, W.SKIP], dtype=np.int32)
    params = [{}] * n_dense + [{"half_width": diag_w}, {"half_width": 60, "offsets": tuple(i * (L // 3) for i in (-2, -1, 0, 1, 2))},
                               {"cols": tuple(range(1, L, 7))}, {}]
    return W.Workload("large-tile", -1, B, n_dense + 4, L, 64, L, 1, 0, table, params, 81)


def cut_text_layer():
    """Long text rows (903 key tiles) over heads whose other items are short: eight waves, and the text items are cut."""
    T = 256
    return W.Workload("cut-text", -1, 1, 4, 115456, 64, 3600, 32, T, np.asarray([W.DIAG] * 4, dtype=np.int32),
                      [{"half_width": 3500, "text_tokens": T}] * 4, 82)


def test_full_size_tables(replay, tmp_path):
    """The two longest benchmark layers keep their other forms in bf16; long D = 64 layers of 400 to 2,500 key tiles per
    resident work-group take the large query tile, some of them with cut items."""
    layers = [layer_text(W.cogvideox15(), 0, rounds=1, tensors=0), layer_text(W.wan21(), 0, rounds=1, tensors=0)]
    res = run(replay, tmp_path, layers)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    assert tables_of(res) == set()
    res = run(replay, tmp_path, [layer_text(large_tile_layer(20011, 9, 5000), 0, rounds=1, tensors=0)])
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    assert tables_of(res) == {(8, False)}
    res = run(replay, tmp_path, [layer_text(cut_text_layer(), 0, rounds=1, tensors=0)])
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    assert tables_of(res) == {(8, True)}


def test_eight_wave_table_stores_every_row_once(replay, tmp_path):
    """The large query tile with the tensors checked (four compute units make a small layer long)."""
    res = run(replay, tmp_path, [layer_text(large_tile_layer(5003, n, 1500), 0, rounds=1, cu=4) for n in (8, 12)])
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    assert tables_of(res) == {(8, False)}


def mixed_layer(D, n_dense, n_diag, n_multi, n_stripe, frame_tokens, frames):
    n, L = frame_tokens, frame_tokens * frames
    table = np.asarray([W.DENSE] * n_dense + [W.DIAG] * n_diag + [W.MULTIDIAG] * n_multi + [W.VSTRIPE] * n_stripe, dtype=np.int32)
    params = [{}] * n_dense + [{"half_width": n}] * n_diag + [{"half_width": n // 4, "offsets": (-2 * n, -n, 0, n, 2 * n)}] * n_multi \
        + [{"cols": tuple(range(0, L, L // 2000))}] * n_stripe
    return W.Workload("mixed", -1, 1, len(table), L, D, n, frames, 0, table, params, 83)


@pytest.mark.parametrize("shape,waves", [
    ((128, 2, 16, 10, 10, 1560, 21), 4),     # a third of the tiles dense
    ((128, 18, 9, 6, 6, 900, 12), 4),        # four fifths, 505 dense tiles per resident work-group
    ((128, 18, 9, 6, 6, 1000, 14), 0),       # 830: the layer kernel
    ((128, 0, 20, 10, 10, 2100, 21), 4),     # none
    ((128, 0, 20, 10, 10, 2100, 33), 0),     # over 2,500 tiles
    ((128, 1, 2, 1, 0, 1600, 24), 0),        # 300 long items in 512 slots: 1.3 times the even load
    ((64, 1, 2, 1, 0, 2000, 33), 0),         # 258 long items in 256 slots
    ((64, 1, 2, 1, 0, 2000, 32), 8),         # 250
    ((64, 1, 2, 1, 0, 1600, 24), 4)])        # uneven, but short
def test_which_layers_run_from_a_table(replay, tmp_path, shape, waves):
    """Both sides of each line of the rule, with 256 compute units."""
    res = run(replay, tmp_path, [layer_text(mixed_layer(*shape), 0, rounds=1, tensors=0)])
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    assert f"layer mixed: table waves {waves}," in res.stdout, res.stdout


@pytest.mark.parametrize("shape,cut", [
    ((64, 2, 3, 1, 1, 1000, 20), True),      # long items three quarters of the layer, a quarter above the share: halved
    ((64, 1, 8, 4, 4, 1000, 20), False),     # two fifths: whole
    ((64, 2, 3, 1, 1, 600, 20), False),      # under 100 tiles a slot: whole up to twice the share
    ((128, 2, 3, 1, 1, 1000, 20), True),
    ((128, 1, 3, 1, 1, 1500, 20), False)])   # two thirds: whole, though 1.5 times the share
def test_which_long_items_are_halved(replay, tmp_path, shape, cut):
    """Both sides of the rule that cuts items above an even share, with 256 compute units."""
    res = run(replay, tmp_path, [layer_text(mixed_layer(*shape), 0, rounds=1, tensors=0)])
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    first = next(line.split() for line in res.stdout.splitlines() if line.startswith("grid:"))   # (the last one is of a rotated table)
    assert (int(first[2]), int(first[6]) > 0) == (4, cut), res.stdout


@pytest.mark.parametrize("shape,items,chunks", [
    ((64, 2, 3, 1, 1, 1000, 20), 314, 2),     # long items of 1.3 shares, three quarters of the layer: halved
    ((128, 2, 3, 1, 1, 1000, 20), 314, 2),
    ((64, 1, 8, 4, 4, 1000, 20), 0, 0),       # two fifths of the layer: whole
    ((64, 2, 3, 1, 1, 600, 20), 0, 0),        # under 100 tiles a slot: whole up to twice the share
    ((128, 1, 3, 1, 1, 1500, 20), 0, 0),      # two thirds of the layer: whole, though 1.5 times the share
    ((128, 5, 8, 0, 0, 470, 20), 0, 0),       # 1.1 shares: whole
    ((128, 2, 2, 0, 3, 750, 20), 236, 2),     # 1.8 shares: two pieces, not three
    ((128, 2, 3, 0, 6, 715, 20), 0, 0),       # 1.9 shares, but 224 items: a compute unit for each
    ((128, 1, 2, 0, 0, 1200, 20), 188, 2),    # 2.2 shares: two pieces of 1.1, as without the rule
    ((128, 1, 1, 0, 0, 1100, 20), 172, 4),    # 2.6 shares: the two pieces of 1.3 halved
    ((128, 1, 2, 0, 0, 1550, 20), 243, 2)])   # 1.7 shares, 243 items
def test_into_how_many_pieces_long_items_are_cut(replay, tmp_path, shape, items, chunks):
    """Both sides of the rule that halves long items, with 256 compute units: how many are cut, and into how many pieces."""
    res = run(replay, tmp_path, [layer_text(mixed_layer(*shape), 0, rounds=1, tensors=0)])
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    first = next(line.split() for line in res.stdout.splitlines() if line.startswith("grid:"))   # (the last one is of a rotated table)
    assert (int(first[2]), int(first[6]), int(first[10])) == (4, items, items * chunks), res.stdout
    assert int(first[10]) <= 1.5 * 512


@pytest.mark.parametrize("shape,waves,items", [
    ((128, 1, 3, 0, 0, 1560, 20), 4, 244),   # three quarters of the layer in 244 long dense items of 1.6 shares: halved
    ((128, 1, 4, 0, 0, 1560, 20), 0, 0),     # 0.7 of it: they would stay whole, more than 30 to an XCD
    ((128, 1, 4, 0, 0, 1536, 20), 4, 0),     # 240 items, 30 to an XCD: whole
    ((128, 1, 2, 0, 0, 1920, 20), 0, 0),     # over 400 tiles a slot
    ((128, 1, 3, 0, 0, 1500, 20), 4, 235)])  # under 300
def test_long_uneven_dense_items_are_halved_or_leave_the_table(replay, tmp_path, shape, waves, items):
    """Both sides of each line of the rule at D = 128 between 300 and 400 tiles a slot, with 256 compute units."""
    res = run(replay, tmp_path, [layer_text(mixed_layer(*shape), 0, rounds=1, tensors=0)])
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    assert f"layer mixed: table waves {waves}," in res.stdout, res.stdout
    if waves:
        first = next(line.split() for line in res.stdout.splitlines() if line.startswith("grid:"))
        assert (int(first[6]), int(first[10])) == (items, 2 * items), res.stdout


def test_a_table_that_cannot_be_built_leaves_no_trace(tmp_path):
    exe = str(tmp_path / "grid_table_fails")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", STUB, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(CSRC, "pattern_compiler.cpp"), os.path.join(STUB, "grid_table_fails.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, (res.returncode, res.stdout)


def test_a_workspace_without_room_for_an_optional_table(tmp_path):
    exe = str(tmp_path / "small_workspace")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
           "-fno-sanitize-recover=undefined", "-I", STUB, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(CSRC, "api.cpp"), os.path.join(CSRC, "pattern_compiler.cpp"),
           *(os.path.join(STUB, f) for f in ("hip_stub.cpp", "launch_models.cpp", "grid_model.cpp", "small_workspace.cpp")), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]


def test_a_long_plan_is_compiled_in_memory_reserved_once(tmp_path):
    exe = str(tmp_path / "plan_memory")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", STUB, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(CSRC, "pattern_compiler.cpp"), os.path.join(STUB, "plan_memory.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, (res.returncode, res.stdout)


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("mode", [W.DENSE, W.DIAG, W.MULTIDIAG, W.VSTRIPE])
def test_cut_items_of_every_kind(D, mode):
    """One head of one mode on a length that gives few query tiles: each is cut into chunks of a few key tiles, among
    them band chunks in which some rows keep no key; keys whose logits rise make the chunks' references differ."""
    L = 1930
    table = np.asarray([mode], dtype=np.int32)
    p = {W.DENSE: {}, W.DIAG: {"half_width": 700}, W.MULTIDIAG: {"half_width": 90, "offsets": (-1500, -600, 0, 640, 1400)},
         W.VSTRIPE: {"cols": tuple(range(5, L, 2))}}[mode]
    wl = W.Workload("cut", -1, 1, 1, L, D, 386, 5, 0, table, [p], 77)
    q, k, v = (t.to("cuda:0") for t in W.make_qkv(wl))
    # Up to twice N(0, 1): the specified arithmetic (bf16 pre-scaled Q, bf16 P, bf16 output, all else exact), carried out
    # on the CPU, is off by at most 1.01e-2 here, inside the bar of 2e-2; with keys up to three times N(0, 1) it is off by
    # 2.2e-2 by itself.
    k = (k * torch.linspace(0.2, 2.0, L, device="cuda:0")[:, None]).to(torch.bfloat16)
    out = run_planned(wl, q, k, v)
    check_layer(wl, q, k, v, out)
    out8, _ = run_fp8(wl, q, k, v)
    check_layer_fp8(wl, q, k, v, out8)


@pytest.mark.gpu
@pytest.mark.parametrize("wl,rows", [(large_tile_layer(20011, 9, 5000), (0, 1, 255, 256, 4999, 5000, 10005, 19967, 19968, 20010)),
                                     (cut_text_layer(), (0, 127, 128, 255, 256, 257, 3755, 57728, 115455))],
                         ids=["ragged", "cut-text"])
def test_eight_wave_table(wl, rows):
    """Layers of 400 to 2,500 key tiles per resident work-group at D = 64 run on the large query tile: a ragged one with
    lists appended for it, and one whose text rows are cut into chunks and merged."""
    gen = torch.Generator(device="cuda:0").manual_seed(wl.seed)
    q, k, v = (torch.randn(wl.B, wl.H, wl.L, wl.D, generator=gen, device="cuda:0", dtype=torch.bfloat16) for _ in range(3))
    desc = svd.desc_of(q)
    ws = torch.empty(svd.svd_plan_workspace_bytes(desc, wl.strategy_table, wl.pattern_params), dtype=torch.uint8, device="cuda:0")
    plan = svd.svd_plan_create(desc, wl.strategy_table, wl.pattern_params, workspace=ws)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert plan.table()["bf16"] == 8
    out = torch.full_like(q, float("nan"))
    svd.svd_attn_forward_planned(plan, q, k, v, out)
    torch.cuda.synchronize()
    plan.close()
    assert torch.isfinite(out).all()
    check_layer(wl, q, k, v, out, rows=np.asarray(rows))


@pytest.mark.gpu
@pytest.mark.parametrize("D,n_cols", [(64, 65), (64, 129), (128, 1), (128, 130)])
def test_padding_of_the_column_list_reads_no_key(D, n_cols):
    """A stripe head whose list ends inside a key tile: the rows that fill the tile are not rows of the tensor, so a NaN
    in a key outside the list (row 0 among them) reaches no output."""
    L = 700
    cols = tuple(range(3, 3 + n_cols))
    wl = W.Workload("pad", -1, 1, 2, L, D, 140, 5, 0, np.asarray([W.VSTRIPE, W.DIAG], dtype=np.int32),
                    [{"cols": cols}, {"half_width": 40}], 78)
    q, k, v = (t.to("cuda:0") for t in W.make_qkv(wl))
    k2, v2 = k.clone(), v.clone()
    outside = [r for r in range(L) if r not in cols]
    k2[:, 0, outside] = float("nan")
    v2[:, 0, outside] = float("nan")
    out = run_planned(wl, q, k2, v2)
    check_layer(wl, q, k, v, out)


@pytest.mark.gpu
@pytest.mark.parametrize("L,D,H", [(1, 64, 2), (128, 128, 3), (129, 64, 3), (257, 128, 2), (1000, 64, 6), (4333, 128, 16)])
def test_dense_entry_point_on_the_small_tile(L, D, H):
    """Few work-groups, or a last round of large ones left nearly empty (4,333 x 16): the dense call takes the small
    query tile; the bits are those of the large one (svd_plan with single_launch = 2, dense_split = 1)."""
    wl = W.small(L=L, D=D, H=H, seed=21)
    wl.strategy_table[:] = W.DENSE
    q, k, v = (t.to("cuda:0") for t in W.make_qkv(wl))
    out = torch.full_like(q, float("nan"))
    svd.svd_dense_attn_forward(q, k, v, out)
    desc = svd.desc_of(q)
    opt = dict(single_launch=2, dense_split=1)
    ws = torch.empty(svd.svd_plan_workspace_bytes(desc, wl.strategy_table, wl.pattern_params, **opt), dtype=torch.uint8, device="cuda:0")
    plan = svd.svd_plan_create(desc, wl.strategy_table, wl.pattern_params, workspace=ws, **opt)
    large = torch.full_like(q, float("nan"))
    svd.svd_attn_forward_planned(plan, q, k, v, large)
    torch.cuda.synchronize()
    plan.close()
    assert torch.equal(out.view(torch.int16), large.view(torch.int16))
    check_layer(wl, q, k, v, out, heads=[0], rows=None if L < 2000 else np.arange(0, L, 97))


@pytest.mark.gpu
@pytest.mark.parametrize("low", [float("-inf"), torch.finfo(torch.bfloat16).min])
@pytest.mark.parametrize("D,mode,options", [
    (64, W.DENSE, {}), (128, W.DENSE, {}), (64, W.VSTRIPE, {}), (128, W.VSTRIPE, {}), (128, W.DIAG, {}), (64, W.MULTIDIAG, {}),
    (64, W.DENSE, {"single_launch": 2, "dense_split": 4}), (128, W.DENSE, {"single_launch": 2, "dense_split": 4})])
def test_a_chunk_of_minus_infinite_logits(D, mode, options, low):
    """Keys masked with the type's lowest value or -inf: the first quarter of the keys has a logit of -inf for every
    query, all others lie some 230 binary orders below zero.  A chunk that holds masked keys alone has no reference; taken
    as one of 0, it would scale every other chunk's results to nothing."""
    L = 1930
    p = {W.DENSE: {}, W.DIAG: {"half_width": 700}, W.MULTIDIAG: {"half_width": 90, "offsets": (-1500, -600, 0, 640, 1400)},
         W.VSTRIPE: {"cols": tuple(range(5, L, 2))}}[mode]
    wl = W.Workload("masked", -1, 1, 1, L, D, 386, 5, 0, np.asarray([mode], dtype=np.int32), [p], 79)
    q, k, v = (t.to("cuda:0") for t in W.make_qkv(wl))
    # logits: D * 1 * -20 * (64 / D) / sqrt(D) * log2(e), about -230 (D = 64) and -163 (D = 128), and a spread of about one
    # around that from the small random part (the common offset cancels in the softmax, its rounding with it)
    q = (1.0 + 0.05 * q.float().clamp(-3, 3)).to(torch.bfloat16)
    k = (-20.0 * 64 / D + 0.3 * k.float()).to(torch.bfloat16)
    k[:, :, :480] = low
    desc = svd.desc_of(q)
    ws = torch.empty(svd.svd_plan_workspace_bytes(desc, wl.strategy_table, wl.pattern_params, **options), dtype=torch.uint8, device="cuda:0")
    plan = svd.svd_plan_create(desc, wl.strategy_table, wl.pattern_params, workspace=ws, **options)
    out = torch.full_like(q, float("nan"))
    svd.svd_attn_forward_planned(plan, q, k, v, out)
    torch.cuda.synchronize()
    plan.close()
    check_layer(wl, q, k, v, out)

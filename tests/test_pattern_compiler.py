"""Host-side checks of the C-ABI library that need no GPU: the shared library
loads and exports what the header declares, argument validation, and the pattern
compiler's lists bit-exact against the oracle's explicit-mask lists."""
import json
import os
import re

import numpy as np
import pytest

from oracle import sparse_attention as O
from paper_2506_03065_amd import binding as svd
from paper_2506_03065_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GOLDEN = json.load(open(os.path.join(ROOT, "tests", "golden", "pattern_counts.json")))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "sparse_vdit.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(svd_[a-z0-9_]+|sparse_vdit_attn_forward[a-z_]*)\s*\(", header))
    assert declared == set(svd.EXPORTS)
    lib = svd.lib()
    for name in declared:
        assert getattr(lib, name) is not None
    assert svd.status_string(0) == "ok"
    assert svd.svd_default_blocks(64)[0] > 0 and svd.svd_default_blocks(128)[1] > 0


def _compile(wl, bq, bk):
    desc = svd.tensor_desc(wl.B, wl.H, wl.L, wl.D)
    return svd.svd_plan_create(desc, wl.strategy_table, wl.pattern_params, bq, bk)


def _assert_plan_matches_oracle(wl, bq, bk, q_blocks=None, plan=None):
    """plan = None: compiled here with the explicit shape bq x bk.  A given plan (for instance one compiled with
    the library's defaults) is checked group by group on the query tile the group reports; q_blocks may then be
    a function of the number of query blocks."""
    plan = _compile(wl, bq, bk) if plan is None else plan
    got_groups = plan.groups()
    want_groups = O.head_groups(wl.strategy_table, wl.pattern_params)
    assert [(g["mode"], g["heads"], g["list_id"], g["rearranged"]) for g in got_groups] == \
           [(g["mode"], g["heads"], g["list_id"], g["rearranged"]) for g in want_groups]
    for gi, g in enumerate(got_groups):
        if g["mode"] in (svd.SVD_DENSE, svd.SVD_SKIP):
            assert g["n_lists"] == 0
            continue
        assert g["n_lists"] == want_groups[gi]["n_lists"]
        for lst in range(g["n_lists"]):
            head = g["heads"][g["list_id"].index(lst)]
            p = wl.pattern_params[head]
            if g["mode"] == svd.SVD_VSTRIPE:
                got = plan.column_list(gi, lst)
                want = O.column_list(p, wl.L, bk)
                assert got["n_cols"] == len(set(p["cols"]) | set(range(O.text_tokens_of(p))))
                assert got["cols"].dtype == np.int32 and np.array_equal(got["cols"], want)
                continue
            got = plan.band_list(gi, lst)
            bq = g["block_q"]
            assert g["block_k"] == bk
            if g["rearranged"]:
                got["row_map"] = plan.row_map(gi, lst)
                want = O.block_lists(g["mode"], p, wl.L, bq, bk)
                assert np.array_equal(got["row_map"], want["row_map"]) and got["row_map"].dtype == np.int32
            if q_blocks is None:
                want = O.block_lists(g["mode"], p, wl.L, bq, bk)
                for key in ("row_ptr", "kv_block_idx", "flags", "run_first", "run_count", "runs"):
                    assert got[key].dtype == np.int32
                    assert np.array_equal(got[key], want[key]), (wl.name, g["mode"], key)
            else:
                runs = O.delta_runs(g["mode"], p, wl.L)
                assert np.array_equal(got["runs"], runs)
                assert got["row_ptr"].size == -(-wl.L // bq) + 1
                for qb in (q_blocks(-(-wl.L // bq)) if callable(q_blocks) else q_blocks):
                    kb, fl, rf, rc = O.query_block_entries(g["mode"], p, wl.L, bq, bk, qb, runs)
                    s, e = got["row_ptr"][qb], got["row_ptr"][qb + 1]
                    assert np.array_equal(got["kv_block_idx"][s:e], kb), (wl.name, qb)
                    assert np.array_equal(got["flags"][s:e], fl), (wl.name, qb)
                    assert np.array_equal(got["run_first"][s:e], rf)
                    assert np.array_equal(got["run_count"][s:e], rc)
    plan.close()


@pytest.mark.parametrize("bq,bk", [(128, 128), (64, 64), (256, 64), (256, 128), (32, 16)])
def test_tiny_lists_bit_exact(bq, bk):
    _assert_plan_matches_oracle(W.tiny(), bq, bk)


@pytest.mark.parametrize("L,D,seed", [(333, 64, 7), (200, 128, 11), (1000, 64, 3), (77, 128, 5)])
@pytest.mark.parametrize("bq,bk", [(256, 64), (256, 128), (16, 8), (7, 5)])
def test_small_ragged_lists_bit_exact(L, D, seed, bq, bk):
    _assert_plan_matches_oracle(W.small(L=L, D=D, seed=seed), bq, bk)


def _one_head(mode, p, L):
    from paper_2506_03065_amd.workloads import Workload
    base = {"half_width": 0, "offsets": (), "cols": ()}
    base.update(p)
    return Workload("adhoc", -1, 1, 1, L, 64, L, 1, 0, np.asarray([mode], dtype=np.int32), [base], 1)


@pytest.mark.parametrize("mode,p,L,bq,bk", [
    (O.MODE_MULTIDIAG, {"half_width": 3, "offsets": (0, 7, -7, 30)}, 47, 16, 4),     # touching bands merge
    (O.MODE_MULTIDIAG, {"half_width": 1, "offsets": (0, 4, 9)}, 40, 8, 16),          # several runs per tile
    (O.MODE_MULTIDIAG, {"half_width": 2, "offsets": (0, 5, 11, 17, 23)}, 90, 32, 32),
    (O.MODE_MULTIDIAG, {"half_width": 0, "offsets": (0, -100, 100)}, 33, 4, 8),      # bands off the map
    (O.MODE_MULTIDIAG, {"half_width": 4, "offsets": (-20, 20, 0)}, 64, 64, 64),      # one tile in all
    (O.MODE_DIAG, {"half_width": 1000}, 130, 64, 32),                                # wider than the map
    (O.MODE_DIAG, {"half_width": 0}, 130, 64, 32),
])
def test_band_edge_cases_bit_exact(mode, p, L, bq, bk):
    _assert_plan_matches_oracle(_one_head(mode, p, L), bq, bk)


@pytest.mark.parametrize("name", ["cogvideox1.5", "hunyuanvideo", "wan2.1"])
def test_full_size_counts_and_sampled_blocks(name):
    """At the benchmark shapes: listed-tile counts equal the stored counts, the
    element counts equal the closed form, and sampled query blocks (first, last,
    around a frame boundary) equal the oracle's explicit-mask entries."""
    wl = W.BY_NAME[name]()
    g = GOLDEN[name]
    for bs, key in ((128, "tiles128"), (64, "tiles64")):
        plan = _compile(wl, bs, bs)
        for gi, grp in enumerate(plan.groups()):
            if grp["mode"] == svd.SVD_DIAG:
                assert plan.band_list(gi, 0)["kv_block_idx"].size == g[key]["diag"]
            if grp["mode"] == svd.SVD_MULTIDIAG:
                assert plan.band_list(gi, 0)["kv_block_idx"].size == g[key]["multi"]
        plan.close()
    bq, bk = svd.svd_default_blocks(wl.D)
    plan = _compile(wl, bq, bk)
    counts = {int(m): int((wl.strategy_table == m).sum()) for m in range(5)}
    want_pairs = (counts[0] * wl.L ** 2 + counts[2] * g["diag"]["pairs"] + counts[3] * g["multi"]["pairs"] +
                  counts[4] * g["vertical"]["pairs"])
    assert plan.work()["kept_pairs"] == float(want_pairs)
    plan.close()
    n_qb = -(-wl.L // bq)
    frame_edge = (wl.text_tokens + 3 * wl.frame_tokens) // bq
    _assert_plan_matches_oracle(wl, bq, bk, q_blocks=[0, frame_edge, n_qb - 1])


def test_work_counts_tiny():
    wl = W.tiny()
    plan = _compile(wl, 128, 128)
    w = plan.work()
    g = GOLDEN["tiny"]
    assert w["kept_pairs"] == 1024 * 1024 + g["diag"]["pairs"] + g["multi"]["pairs"] + g["vertical"]["pairs"]
    assert w["computed_tiles"] == 64 + g["tiles128"]["diag"] + g["tiles128"]["multi"] + 8 * 1
    assert w["computed_flops"] == 4.0 * 64 * (1024 * 1024 + (22 + 44) * 128 * 128 + 1024 * 64)


def _status(fn, *a, **kw):
    try:
        fn(*a, **kw)
    except svd.SvdError as e:
        return e.status
    return 0


def test_validation_errors():
    d = svd.tensor_desc(1, 2, 100, 64)
    ok = [{"half_width": 3}, {"cols": (1, 2)}]
    mk = lambda table, params, desc=d: _status(svd.svd_plan_create, desc, table, params)
    assert mk([2, 4], ok) == 0
    assert mk([2, 5], ok) == 5                                              # mode id
    assert mk([2, -1], ok) == 5
    assert mk([2, 4], [{"half_width": -1}, ok[1]]) == 6                    # negative width
    assert mk([3, 4], [{"half_width": 1, "offsets": ()}, ok[1]]) == 6      # no offsets
    assert mk([3, 4], [{"half_width": 1, "offsets": (0, 5, 5)}, ok[1]]) == 6   # duplicate offsets
    assert mk([3, 4], [{"half_width": 1, "offsets": (6,)}, ok[1]]) == 7    # first rows keep nothing
    assert mk([3, 4], [{"half_width": 1, "offsets": (-6, 6)}, ok[1]]) == 0     # every row keeps a key
    assert mk([2, 4], [ok[0], {"cols": ()}]) == 7                          # no columns
    assert mk([2, 4], [ok[0], {"cols": (1, 1)}]) == 6                      # duplicate column
    assert mk([2, 4], [ok[0], {"cols": (100,)}]) == 6                      # column out of range
    assert mk([2, 4], [ok[0], {"cols": (-1,)}]) == 6
    assert mk([0, 0], ok, svd.tensor_desc(1, 2, 100, 96)) == 2             # head dim
    assert mk([0, 0], ok, svd.tensor_desc(1, 2, 0, 64)) == 2               # empty sequence
    assert mk([0, 0], ok, svd.tensor_desc(1, 2, 100, 64, stride_l=68)) == 4   # row alignment
    assert mk([0, 0], ok, svd.tensor_desc(1, 2, 100, 64, stride_l=32)) == 2
    # size limits: 32-bit byte offsets inside a head, 24-bit row index and row stride
    assert _status(svd.svd_plan_workspace_bytes, svd.tensor_desc(1, 2, 1 << 22, 64, stride_l=512), [0, 0], ok) == 9
    assert _status(svd.svd_plan_workspace_bytes, svd.tensor_desc(1, 2, 100, 64, stride_l=1 << 23), [0, 0], ok) == 9
    assert _status(svd.svd_plan_workspace_bytes, svd.tensor_desc(1, 2, 100, 64, stride_l=(1 << 23) - 8), [0, 0], ok) == 0
    assert _status(svd.svd_plan_workspace_bytes, d, [2, 9], ok) == 5
    assert svd.svd_plan_workspace_bytes(d, [2, 4], ok) > 0
    with pytest.raises(svd.SvdError):
        svd.svd_default_blocks(96)


def test_host_only_plan_refuses_to_launch():
    wl = W.tiny()
    plan = _compile(wl, 0, 0)
    import ctypes
    st = svd.lib().svd_attn_forward_planned(plan.handle, ctypes.c_void_p(16), ctypes.c_void_p(16),
                                            ctypes.c_void_p(16), ctypes.c_void_p(16), None)
    assert st == 8
    st = svd.lib().svd_attn_forward_planned(plan.handle, None, None, None, None, None)
    assert st == 1
    st = svd.lib().svd_attn_forward_planned(plan.handle, ctypes.c_void_p(8), ctypes.c_void_p(16),
                                            ctypes.c_void_p(16), ctypes.c_void_p(16), None)
    assert st == 4


def test_workspace_holds_lists_and_the_scratch_of_a_forced_dense_split():
    """With dense_split forced the workspace is the list image, padded to 256
    bytes, plus per chunk item and wave (D/2 + 2) rows of 64 floats."""
    wl = W.small(L=1000, D=64, H=5, seed=3, B=2)
    desc = svd.tensor_desc(wl.B, wl.H, wl.L, wl.D)
    base = svd.svd_plan_workspace_bytes(desc, wl.strategy_table, wl.pattern_params, dense_split=1)
    n_dense = int((wl.strategy_table == 0).sum())
    bq, bk = svd.svd_default_blocks(wl.D)
    for split in (2, 3, 8):
        got = svd.svd_plan_workspace_bytes(desc, wl.strategy_table, wl.pattern_params, dense_split=split)
        chunks = min(split, -(-wl.L // bk))
        items = -(-wl.L // bq) * n_dense * wl.B * chunks
        waves = bq // 32
        want = -(-base // 256) * 256 + items * waves * (wl.D // 2 + 2) * 64 * 4
        assert got == (want if n_dense else base)
    with pytest.raises(svd.SvdError):
        svd.svd_plan_workspace_bytes(desc, wl.strategy_table, wl.pattern_params, dense_split=-1)


# ---- text prefix (Section 4.1.1): borders kept whole by the sparse heads ----

@pytest.mark.parametrize("L,D,seed,bq,bk,T", [(600, 64, 7, 64, 32, 64), (1000, 128, 3, 256, 64, 256),
                                               (1000, 64, 4, 256, 128, 256), (333, 64, 5, 16, 8, 32),
                                               (700, 128, 6, 256, 64, 512)])
def test_text_prefix_lists_bit_exact(L, D, seed, bq, bk, T):
    wl = W.with_text_borders(W.small(L=L, D=D, H=10, seed=seed), T)
    _assert_plan_matches_oracle(wl, bq, bk)


@pytest.mark.parametrize("mode,p,L,bq,bk", [
    (O.MODE_DIAG, {"half_width": 0, "text_tokens": 16}, 130, 16, 8),                       # band never reaches the text
    (O.MODE_DIAG, {"half_width": 1000, "text_tokens": 16}, 130, 16, 16),                   # band covers everything
    (O.MODE_MULTIDIAG, {"half_width": 2, "offsets": (-40, 0, 40), "text_tokens": 32}, 150, 32, 8),
    (O.MODE_MULTIDIAG, {"half_width": 1, "offsets": (50,), "text_tokens": 8}, 60, 8, 8),   # rows that keep text keys only
])
def test_text_prefix_band_edge_cases_bit_exact(mode, p, L, bq, bk):
    _assert_plan_matches_oracle(_one_head(mode, p, L), bq, bk)


def test_text_prefix_counts_and_validation():
    L, T = 1000, 256
    wl = W.with_text_borders(W.small(L=L, D=64, H=5, seed=9), T)
    plan = _compile(wl, 256, 128)
    # element-level sparsity against the explicit mask
    sp = plan.head_sparsity()
    for h in range(wl.H):
        mode, p = int(wl.strategy_table[h]), wl.pattern_params[h]
        want = 0.0 if mode == W.DENSE else 1.0 if mode == W.SKIP else 1.0 - O.mask_popcount(mode, p, L) / L ** 2
        assert abs(sp[h] - want) < 1e-12, (h, mode)
    # computed tiles: the lists plus one dense query tile of text rows per sparse head
    n_kb = -(-L // 128)
    want_tiles = n_kb * -(-L // 256)                                  # the dense head
    for h in range(wl.H):
        mode, p = int(wl.strategy_table[h]), wl.pattern_params[h]
        if mode in O.BAND_MODES:
            want_tiles += O.block_lists(mode, p, L, 256, 128)["kv_block_idx"].size + (T // 256) * n_kb
        elif mode == W.VSTRIPE:
            want_tiles += -(-L // 256) * (O.column_list(p, L, 128).size // 128) + (T // 256) * n_kb
    assert plan.work()["computed_tiles"] == want_tiles
    plan.close()
    desc = svd.tensor_desc(1, wl.H, L, 64)
    for T_bad, status in ((100, 9), (128, 9), (1024, 6), (-256, 6)):   # not a multiple of both blocks; not shorter than L
        with pytest.raises(svd.SvdError) as e:
            svd.svd_plan_create(desc, wl.strategy_table, wl.pattern_params, 256, 128, text_tokens=T_bad)
        assert e.value.status == status, T_bad
    mixed = [dict(p) for p in wl.pattern_params]
    mixed[1]["text_tokens"] = 512
    with pytest.raises(ValueError):
        svd.svd_plan_create(desc, wl.strategy_table, mixed, 256, 128)
    # a pattern that leaves rows without band keys is accepted once they keep the text keys
    lonely = W.with_text_borders(_one_head(O.MODE_MULTIDIAG, {"half_width": 1, "offsets": (50,)}, 600), 256)
    _compile(lonely, 256, 128).close()
    with pytest.raises(svd.SvdError) as e:
        _compile(_one_head(O.MODE_MULTIDIAG, {"half_width": 1, "offsets": (50,)}, 600), 256, 128)
    assert e.value.status == 7


# ---- multi-diagonal heads in rearranged form (Section 4.1.2) ----

@pytest.mark.parametrize("L,bq,bk,first,N,F,w", [(600, 64, 32, 0, 60, 10, 25), (1000, 256, 64, 40, 96, 10, 50),
                                                  (333, 16, 8, 13, 32, 10, 0), (1000, 256, 128, 0, 1000, 1, 7)])
def test_rearranged_heads_lists_and_row_map_bit_exact(L, bq, bk, first, N, F, w):
    wl = W.small(L=L, D=64, H=10, seed=3)
    params = [dict(p) for p in wl.pattern_params]
    multi = [h for h in range(wl.H) if wl.strategy_table[h] == W.MULTIDIAG]
    params[multi[0]] = {"half_width": w, "offsets": (), "cols": (), "rearranged": (first, N, F)}
    wl.pattern_params = params
    _assert_plan_matches_oracle(wl, bq, bk)
    plan = _compile(wl, bq, bk)
    groups = plan.groups()
    assert [g["rearranged"] for g in groups if g["mode"] == W.MULTIDIAG] == [False, True]
    sp = plan.head_sparsity()
    assert abs(sp[multi[0]] - (1.0 - O.mask_popcount(W.MULTIDIAG, params[multi[0]], L) / L ** 2)) < 1e-12
    plan.close()


def test_rearranged_heads_validation():
    desc = svd.tensor_desc(1, 1, 512, 64)
    table = [W.MULTIDIAG]
    for geo, status in (((0, 100, 6), 6), ((-1, 10, 4), 6), ((0, 0, 4), 6), ((500, 4, 4), 6)):
        with pytest.raises(svd.SvdError) as e:
            svd.svd_plan_create(desc, table, [{"half_width": 3, "rearranged": geo}], 256, 128)
        assert e.value.status == status, geo
    with pytest.raises(svd.SvdError) as e:      # not combined with a text prefix
        svd.svd_plan_create(desc, table, [{"half_width": 3, "rearranged": (256, 64, 4), "text_tokens": 256}], 256, 128)
    assert e.value.status == 9
    with pytest.raises(svd.SvdError) as e:
        svd.svd_plan_create(desc, table, [{"half_width": -1, "rearranged": (0, 64, 4)}], 256, 128)
    assert e.value.status == 6


# ---- small query tile for band groups with narrow bands ----

def test_default_plan_gives_narrow_band_groups_the_small_query_tile():
    L, D = 3000, 64
    table = np.asarray([W.DENSE, W.DIAG, W.MULTIDIAG, W.VSTRIPE, W.MULTIDIAG], dtype=np.int32)
    params = [{}, {"half_width": 2990}, {"half_width": 20, "offsets": (-600, 0, 600)}, {"cols": tuple(range(0, L, 9))},
              {"half_width": 30, "rearranged": (0, 300, 10)}]
    wl = W.Workload("tiles", -1, 1, len(table), L, D, 600, 5, 0, table, params, 3)
    desc = svd.tensor_desc(1, wl.H, L, D)
    plan = svd.svd_plan_create(desc, table, params)                # block shape left to the library
    bq, bk = svd.svd_default_blocks(D)
    small = {g["mode"]: g["block_q"] for g in plan.groups() if not g["rearranged"]}
    assert small[W.DENSE] == bq and small[W.VSTRIPE] == bq
    assert small[W.DIAG] == bq                                      # a band as wide as the map gains nothing
    assert small[W.MULTIDIAG] == bq // 2                            # narrow bands: half the query rows per tile
    for gi, g in enumerate(plan.groups()):
        assert g["block_k"] == bk
        if g["mode"] in (W.DIAG, W.MULTIDIAG):
            if g["rearranged"]:
                assert g["block_q"] == bq // 2
            head = g["heads"][0]
            got = plan.band_list(gi, 0)
            want = O.block_lists(g["mode"], params[head], L, g["block_q"], bk)
            for key in ("row_ptr", "kv_block_idx", "flags", "run_first", "run_count", "runs"):
                assert np.array_equal(got[key], want[key]), (g["mode"], key)
    # the work counts follow the chosen tiles
    area = 0.0
    for gi, g in enumerate(plan.groups()):
        for h in g["heads"]:
            mode, p = int(table[h]), params[h]
            if mode == W.DENSE:
                area += L * L
            elif mode == W.VSTRIPE:
                area += L * len(p["cols"])
            else:
                lists = O.block_lists(mode, p, L, g["block_q"], bk)
                rows = np.diff(lists["row_ptr"])
                for qb, n in enumerate(rows):
                    r = min(L, (qb + 1) * g["block_q"]) - qb * g["block_q"]
                    kbs = lists["kv_block_idx"][lists["row_ptr"][qb]:lists["row_ptr"][qb + 1]]
                    area += sum(r * (min(L, (kb + 1) * bk) - kb * bk) for kb in kbs)
    assert abs(plan.work()["computed_flops"] - 4.0 * D * area) <= 1e-6 * 4.0 * D * area
    plan.close()
    # an explicit block shape applies to every group
    plan = svd.svd_plan_create(desc, table, params, bq, bk)
    assert {g["block_q"] for g in plan.groups()} == {bq}
    plan.close()


_STACK_BAND_LISTS = {}


def _stack_band_lists(plan):
    """{(mode, block_q): band list} of a stack layer's plan (every layer uses one diagonal and one multi-diagonal pattern)."""
    out = {}
    for gi, grp in enumerate(plan.groups()):
        if grp["mode"] in (svd.SVD_DIAG, svd.SVD_MULTIDIAG):
            assert grp["n_lists"] == 1
            out[(grp["mode"], grp["block_q"])] = plan.band_list(gi, 0)
    return out


@pytest.mark.parametrize("layer", range(40))
def test_every_stack_layer_compiles_to_the_oracles_groups_and_lists(layer):
    """All 40 strategy tables of the layer stack (dense share falling from 80 % to 10 % with depth), host only,
    both with the kernels' block shape given explicitly and in the plan the library compiles by default (the query
    tile of the band groups is its choice): mode counts, groups, list ids, every column list and the runs of kept
    diagonals bit-exact against the oracle; element counts against the closed forms.  The band patterns are the
    same in every layer, so the band lists must equal those of the first layer bit for bit, and those are
    compared with the oracle's explicit-mask entries on sampled query blocks."""
    wl = W.stack_layer(layer)
    counts = W.stack_layer_counts(layer)
    assert sum(counts.values()) == wl.H == 40
    assert counts[W.DENSE] == int(round(40 * (0.8 - 0.7 * layer / 39)))
    assert {m: int((wl.strategy_table == m).sum()) for m in range(5)} == {m: counts.get(m, 0) for m in range(5)}
    bq, bk = svd.svd_default_blocks(wl.D)
    first = not _STACK_BAND_LISTS
    sample = (lambda n_qb: [0, (3 * wl.frame_tokens) // -(-wl.L // n_qb), n_qb - 1]) if first else []
    explicit = _compile(wl, bq, bk)
    default = svd.svd_plan_create(svd.tensor_desc(wl.B, wl.H, wl.L, wl.D), wl.strategy_table, wl.pattern_params)
    lists = {**_stack_band_lists(explicit), **_stack_band_lists(default)}
    assert {k[1] for k in lists} <= {bq, 128}                     # the default plan picks the query tile per band group
    if first:
        _STACK_BAND_LISTS.update(lists)
    for key, bl in lists.items():
        for name, arr in bl.items():
            assert np.array_equal(arr, _STACK_BAND_LISTS[key][name]), (layer, key, name)
    g = GOLDEN["wan2.1"]
    want_pairs = (counts[W.DENSE] * wl.L ** 2 + counts[W.DIAG] * g["diag"]["pairs"] +
                  counts[W.MULTIDIAG] * g["multi"]["pairs"] + counts[W.VSTRIPE] * g["vertical"]["pairs"])
    assert default.work()["kept_pairs"] == float(want_pairs) == explicit.work()["kept_pairs"]
    _assert_plan_matches_oracle(wl, bq, bk, q_blocks=sample, plan=explicit)
    _assert_plan_matches_oracle(wl, bq, bk, q_blocks=sample, plan=default)


def test_wide_bands_run_on_the_large_tile_and_keep_small_tile_lists_for_the_fp8_path():
    """A band so wide that the small query tile saves less than 8 % of the listed area: the group is compiled for
    the large tile, and the plan keeps the small-tile lists for the FP8 kernels; their tile count is the oracle's."""
    L, D = 3000, 64
    table = np.asarray([W.DIAG, W.MULTIDIAG, W.DENSE], dtype=np.int32)
    params = [{"half_width": 1200}, {"half_width": 400, "offsets": (-1000, 0, 1000)}, {}]
    desc = svd.tensor_desc(1, 3, L, D)
    plan = svd.svd_plan_create(desc, table, params)
    bq, bk = svd.svd_default_blocks(D)
    groups = plan.groups()
    assert [g["block_q"] for g in groups] == [bq, bq, bq]
    for gi, g in enumerate(groups):
        mode = g["mode"]
        if mode == W.DENSE:
            assert plan.work_fp8(gi)["computed_tiles"] == plan.work(gi)["computed_tiles"]
            continue
        p = params[g["heads"][0]]
        large = O.block_lists(mode, p, L, bq, bk)["kv_block_idx"].size
        small = O.block_lists(mode, p, L, bq // 2, bk)["kv_block_idx"].size
        assert plan.work(gi)["computed_tiles"] == large
        assert plan.work_fp8(gi)["computed_tiles"] == small
        assert plan.work_fp8(gi)["computed_flops"] < plan.work(gi)["computed_flops"] <= plan.work_fp8(gi)["computed_flops"] / 0.92
    assert plan.work_fp8()["computed_tiles"] == sum(plan.work_fp8(gi)["computed_tiles"] for gi in range(len(groups)))
    plan.close()


def test_marshalled_parameters_word_for_word():
    """The svd_head_params array of dicts of every kind: shared dicts and lists, none at all, read-only, strided, converted
    and two-dimensional lists, integers past 32 bits (which wrap)."""
    fixed = np.arange(5, dtype=np.int32)
    fixed.flags.writeable = False
    shared = {"half_width": 7, "offsets": [-3, 0, 3]}
    params = [None, {}, shared, shared, {"cols": fixed}, {"cols": np.arange(20)[::2]}, {"offsets": (), "cols": ()},
              {"half_width": np.int64(5), "offsets": np.array([[1, 2], [3, 4]])}, {"half_width": 2 ** 31 + 5},
              {"half_width": -2 ** 40 - 1, "rearranged": (1, 2, 3)}, {"half_width": 2.7, "cols": np.array([1.0, 2.0])}]
    want = [(0, [], [], (0, 0, 0))] * 2 + [(7, [-3, 0, 3], [], (0, 0, 0))] * 2 + [
        (0, [], list(range(5)), (0, 0, 0)), (0, [], list(range(0, 20, 2)), (0, 0, 0)), (0, [], [], (0, 0, 0)),
        (5, [1, 2, 3, 4], [], (0, 0, 0)), (5 - 2 ** 31, [], [], (0, 0, 0)), (-1, [], [], (1, 2, 3)), (2, [], [1, 2], (0, 0, 0))]
    m = svd._Marshalled([2] * len(params), params)
    got = [(p.half_width, [p.offsets[i] for i in range(p.n_offsets)], [p.cols[i] for i in range(p.n_cols)],
            (p.rearr_first, p.rearr_frame_tokens, p.rearr_frames)) for p in m.params]
    assert got == want and not any(bool(p.offsets) != (p.n_offsets > 0) or bool(p.cols) != (p.n_cols > 0) for p in m.params)
    with pytest.raises(ValueError):
        svd._Marshalled([1, 2], [{}])


@pytest.mark.parametrize("p", [{"offsets": None}, {"cols": None}, {"half_width": 3, "offsets": None, "cols": [1]}, {"offsets": "x"},
                               {"half_width": None}])
def test_parameters_that_are_no_numbers_are_refused(p):
    """A list given as None is not an absent one."""
    with pytest.raises((TypeError, ValueError)):
        svd._Marshalled([2, 2], [{"half_width": 1}, p])

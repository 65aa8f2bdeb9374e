"""The one-shot call's workspace is the caller's between two calls: lists are never taken for valid because an address is
the same.  On the host model of the runtime, and on the GPU with the workspace overwritten in between."""
import os
import subprocess
import threading

import numpy as np
import pytest
import torch

from paper_2506_03065_amd import binding as svd
from paper_2506_03065_amd import workloads as W
from parity_util import check_layer
from test_host_launch_model import CSRC, ROOT, STUB


def test_calls_on_the_host_model(tmp_path):
    exe = str(tmp_path / "one_shot")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
           "-fno-sanitize-recover=undefined", "-I", STUB, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(CSRC, "api.cpp"), os.path.join(CSRC, "pattern_compiler.cpp"),
           *(os.path.join(STUB, f) for f in ("hip_stub.cpp", "launch_models.cpp", "grid_model.cpp", "one_shot.cpp")), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0")   # the cache keeps its plan to the end
    res = subprocess.run([exe, "6"], capture_output=True, text=True, env=env, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
def test_workspace_used_in_between(D):
    """The same call again after its workspace held other bytes, on the same stream and on another, after calls with
    other tables and workspaces: the same bits each time."""
    wl = W.small(L=900, D=D, H=5, seed=31)
    q, k, v = (t.to("cuda:0") for t in W.make_qkv(wl))
    tables = [np.roll(wl.strategy_table, r).astype(np.int32) for r in range(5)]
    params = [[wl.pattern_params[(h - r) % 5] for h in range(5)] for r in range(5)]
    desc = svd.desc_of(q)
    n = max(svd.svd_plan_workspace_bytes(desc, t, p) for t, p in zip(tables, params))
    ws = [torch.empty(n, dtype=torch.uint8, device="cuda:0") for _ in range(2)]

    def call(r, w, stream=None):
        out = torch.full_like(q, float("nan"))
        torch.cuda.synchronize()
        svd.sparse_vdit_attn_forward(q, k, v, tables[r], params[r], out, ws[w], stream=stream)
        torch.cuda.synchronize()
        return out.view(torch.int16)
    want = [call(r, 0) for r in range(5)]
    check_layer(wl, q, k, v, want[0].view(torch.bfloat16))
    side = torch.cuda.Stream()
    for r in (0, 3):
        call(r, 0)
        for fill in (0x7f, 0xff, 0):
            ws[0].fill_(fill)
            assert torch.equal(call(r, 0, side if fill == 0xff else None), want[r])
    outs = []
    for i in range(40):   # nothing waits in between: copies and launches of different plans follow one another
        out = torch.full_like(q, float("nan"))
        svd.sparse_vdit_attn_forward(q, k, v, tables[i % 5], params[i % 5], out, ws[i % 2])
        outs.append(out)
    torch.cuda.synchronize()
    assert all(torch.equal(o.view(torch.int16), want[i % 5]) for i, o in enumerate(outs))


@pytest.mark.gpu
def test_threads_on_streams_of_their_own():
    """Two threads, each with its stream, workspace and tables, in turn through the one cache: the bits of single calls."""
    wl = W.small(L=900, D=64, H=5, seed=32)
    q, k, v = (t.to("cuda:0") for t in W.make_qkv(wl))
    tables = [np.roll(wl.strategy_table, r).astype(np.int32) for r in range(4)]
    params = [[wl.pattern_params[(h - r) % 5] for h in range(5)] for r in range(4)]
    desc = svd.desc_of(q)
    n = max(svd.svd_plan_workspace_bytes(desc, t, p) for t, p in zip(tables, params))
    ws = [torch.empty(n, dtype=torch.uint8, device="cuda:0") for _ in range(2)]
    want = []
    for t, p in zip(tables, params):
        out = torch.full_like(q, float("nan"))
        svd.sparse_vdit_attn_forward(q, k, v, t, p, out, ws[0])
        torch.cuda.synchronize()
        want.append(out.view(torch.int16))
    outs = [[torch.full_like(q, float("nan")) for _ in range(30)] for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()

    def work(i):
        for j, out in enumerate(outs[i]):
            r = 2 * i + (j // 3) % 2
            svd.sparse_vdit_attn_forward(q, k, v, tables[r], params[r], out, ws[i], stream=streams[i])
    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(o.view(torch.int16), want[2 * i + (j // 3) % 2]) for j, o in enumerate(outs[i]))

"""Whole schedules in one call, whose last pair average also writes the composed map and the
grid, against the same schedule step by step (its own gather), bit for bit."""
import numpy as np
import pytest
import torch

import paper_2604_05718_amd as mpm
from paper_2604_05718_amd import api

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
TORCH_DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def tokens(B, N, D, dtype, seed):
    """Clustered tokens, the last image's all equal (every score tied)."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((B, 6, D))[:, rng.integers(0, 6, N)] + 0.3 * rng.standard_normal((B, N, D))
    x[-1] = x[-1, :1]
    return torch.from_numpy(x.astype(np.float32)).to(TORCH_DT[dtype]).to(DEV)


# Rows of one 16-byte piece, one lane group's width and its neighbours, a wave's batch (512
# pieces) and one more; images shorter than, at and past the rows of a workgroup; the least rows
# that keep 8 lanes each, and fewer.
CASES = [("bf16", 3, 33, 8), ("f32", 2, 40, 28), ("bf16", 5, 64, 64), ("bf16", 2, 257, 72), ("f32", 3, 90, 256),
         ("bf16", 9, 130, 520), ("bf16", 8, 1030, 128), ("bf16", 7, 1000, 128), ("f32", 2, 19, 2048),
         ("bf16", 2, 21, 4104), ("bf16", 4, 1, 64), ("f32", 3, 2, 36)]


@pytest.mark.parametrize("window", [None, 2])
@pytest.mark.parametrize("insertions", [1, 2, 3])
@pytest.mark.parametrize("dtype,B,N,D", CASES)
def test_one_call_equals_steps(dtype, B, N, D, insertions, window):
    print(f"one call {dtype} B={B} N={N} D={D} insertions={insertions} window={window}", flush=True)
    x = tokens(B, N, D, dtype, N * 100 + D)
    local = {} if window is None else dict(grid_w=7, window=window)
    one = api.Schedule(B, N, D, x.dtype, insertions=insertions, device=DEV, **local)
    steps = api.Schedule(B, N, D, x.dtype, insertions=insertions, device=DEV, **local)
    for s in (one, steps):  # nothing may be left from before
        s.out.fill_(7.0)
        s.rstar.fill_(-5)
    a = one.run(x)
    b = steps.run(x, marks=[torch.cuda.Event() for _ in range(steps.n_marks())])
    # One workspace for every insertion: run step by step.
    ws = mpm.new_workspace(B, N, DEV)
    shared = mpm.run_schedule(x, insertions=insertions, workspaces=[ws] * insertions, **local)
    fresh = mpm.run_schedule(x, insertions=insertions, **local)
    torch.cuda.synchronize()
    bits = torch.int16 if dtype == "bf16" else torch.int32
    for out, rstar in ((b, steps.rstar), (shared.out, shared.rstar), (fresh.out, fresh.rstar)):
        assert torch.equal(a.view(bits), out.view(bits)) and torch.equal(one.rstar, rstar)
    for s in range(insertions):
        total = int(steps.y_off[s][-1])
        assert torch.equal(one.y_off[s], steps.y_off[s]) and torch.equal(one.map[s], steps.map[s])
        assert torch.equal(one.y[s][:total].view(bits), steps.y[s][:total].view(bits))
        assert torch.equal(fresh.stages[s].y[:total].view(bits), steps.y[s][:total].view(bits))
        if window is not None:
            assert torch.equal(one.y_pos[s][:total], steps.y_pos[s][:total])
            assert torch.equal(fresh.stages[s].y_pos[:total], steps.y_pos[s][:total])

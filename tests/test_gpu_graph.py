"""Fused steps captured into a HIP graph replay exactly like eager launches.

Each rip_preduce call enqueues one kernel launch (two for long steps that mix
far apart unit shapes) whose argument carries the whole step (schedule, optimizer scalars, the handle's pointer-table address)
and does no memset, copy or allocation, so a sequence of steps can be
captured once and replayed.  The graph is replayed several times with the
program's own eager work and synchronizations in between; after every replay
the buffers must equal both an eager run of the same steps and the oracle.
"""
import numpy as np
import pytest

from seedgen import DTYPE_BF16, DTYPE_F32
from seedgen import workloads as wl

from gpu_util import compare, log, oracle_windows, sample_windows

pytestmark = pytest.mark.gpu

# (active, groups) per captured step: grouped and lone updates, a group whose
# members do not all update, a pure P-Reduce of six, and a step of a group of
# eight, which wants few resident waves, beside a pair and two lone updates,
# which want many: one launch while the step is short, two where it is long
STEPS = [
    ([0, 1, 2, 3, 4, 5], [(0, 1, 2), (3, 4)]),
    ([0, 2, 3], [(1, 5), (2, 3)]),
    ([], [(0, 1, 2, 3, 4, 5)]),
    (list(range(12)), [tuple(range(8)), (8, 9)]),
]


SHORT, LONG = 3 * 4096 + 5, 9_000_005   # elements; the last step moves > 1 GiB at LONG


def _workload(dtype, momentum, P=SHORT):
    return wl.Workload(f"graph_{'bf16' if dtype else 'fp32'}_{'mom' if momentum else 'sgd'}",
                       12, [P], dtype, 0.1 if not dtype else 2.0, momentum,
                       0.01, dict(mode=wl.TABLE, table=[[(0, 1)]]), len(STEPS), 7,
                       param_sigma=1.0 if not dtype else 0.05, grad_ring=1)


def _launch_all(rip, h, w, stream):
    for active, groups in STEPS:
        rip.rip_preduce(h, groups, active, lr=w.lr, momentum=w.momentum, stream=stream)
        split = len(groups[0]) == 8 and w.numel == LONG
        assert rip.rip_last_launch_count() == (2 if split else 1)


def _state(st, w, windows):
    def rows(kind):
        return np.stack([np.concatenate([st.window(kind, r, a, b) for a, b in windows])
                         for r in range(w.n)])
    return rows("param"), rows("mom") if w.momentum else None


@pytest.mark.parametrize("dtype,momentum", [(DTYPE_F32, 0.0), (DTYPE_BF16, 0.9)])
@pytest.mark.parametrize("P", [SHORT, LONG])
def test_graph_replays_match_eager_and_oracle(dtype, momentum, P):
    """Whole buffers where the step is short, sampled windows where it is long
    (exact: the method is element-wise)."""
    import torch
    import paper_1909_08029_amd as rip
    torch.cuda.set_device(0)
    w = _workload(dtype, momentum, P)
    windows = [(0, P)] if P == SHORT else sample_windows(P, 12, 4096, 3)
    log(f"case {w.name} P={P}: capture {len(STEPS)} steps, replay 3 times")
    eager = wl.DeviceState(w)
    eager.fill()
    graphed = wl.DeviceState(w)
    graphed.fill()
    he = rip.Replicas(eager.param, eager.grad_sets[0], eager.mom)
    hg = rip.Replicas(graphed.param, graphed.grad_sets[0], graphed.mom)
    torch.cuda.synchronize()

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _launch_all(rip, hg, w, torch.cuda.current_stream())
    torch.cuda.synchronize()
    # capturing records the launches without running them
    p0, _ = _state(graphed, w, windows)
    pe0, _ = _state(eager, w, windows)
    assert np.array_equal(p0, pe0)

    noise = torch.empty(1 << 20, device="cuda")
    schedule = []
    for rep in range(3):
        g.replay()
        noise.normal_()                      # the program's own eager work
        _ = float(noise.sum())               # ... and a synchronization
        _launch_all(rip, he, w, torch.cuda.current_stream())
        torch.cuda.synchronize()
        schedule += STEPS
        pg, vg = _state(graphed, w, windows)
        pe, ve = _state(eager, w, windows)
        view = np.uint16 if dtype == DTYPE_BF16 else np.uint32
        assert np.array_equal(pg.view(view), pe.view(view)), f"replay {rep}: graph != eager"
        if momentum:
            assert np.array_equal(vg.view(view), ve.view(view)), f"replay {rep}: momentum"
        want = oracle_windows(w, schedule, windows)
        po = np.concatenate([p for p, _ in want], axis=1)
        vo = np.concatenate([v for _, v in want], axis=1) if momentum else None
        for r in range(w.n):
            compare(pg[r], po[r], dtype, f"{w.name} replay {rep} param r={r}")
            if momentum:
                compare(vg[r], vo[r], dtype, f"{w.name} replay {rep} mom r={r}")
    del g
    he.close()
    hg.close()

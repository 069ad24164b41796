"""GPU parity of the nano-batched execution (Sec. 3.3): the batch cut into N nano-batches, processed one after
the other through the C ABI, must give the oracle's result of the whole batch for every N (the nano-batch size is
a performance knob); dA_j / dB_j are accumulated over the nano-batches."""
import time

import numpy as np
import pytest

from paper_2602_07263_amd import workloads as wk
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


def _assert_ok(res, label):
    bad = {k: v for k, v in res.items() if not v <= 1.0}
    assert not bad, f"{label}: worst error / tolerance ratios {res}"


def _run_nano(p, n_nano, granule, flags=0, prefill=None):
    import torch
    from paper_2602_07263_amd import tlora
    lp = tlora.LayerProblem.from_numpy(p)
    tdt = torch.bfloat16 if p.dtype == "bf16" else torch.float32
    dY = torch.from_numpy(p.dY).to(device="cuda", dtype=tdt)
    Y, dX, dA, dB = lp.new_outputs()
    Y.fill_(float("nan")); dX.fill_(float("nan"))
    for t in dA + dB:
        t.fill_(float("nan") if prefill is None else prefill)
    lp.fwd_nano(n_nano, granule, Y)
    lp.bwd_nano(n_nano, granule, dY, dX, dA, dB, flags)
    torch.cuda.synchronize()
    return (Y.float().cpu().numpy(), dX.float().cpu().numpy(), [a.cpu().numpy() for a in dA],
            [b.cpu().numpy() for b in dB])


CASES = [
    ("bf16", 384, 640, [1, 12, 256, 40, 130], [300, 17, 700, 1, 520], [0.5, 2.0, 1.0, 4.0, 2.0]),
    ("f32", 96, 72, [3, 8, 0, 5], [40, 0, 33, 130], [2.0, 1.0, 2.0, 0.5]),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("n_nano,granule", [(1, 64), (2, 64), (5, 32), (9, 1), (64, 64)])
def test_results_do_not_depend_on_the_number_of_nano_batches(case, n_nano, granule):
    dtype, d_in, d_out, ranks, tokens, scales = case
    p = wk.generate(wk.custom("nano", dtype, d_in, d_out, ranks, tokens, scales), seed=5)
    Y, dX, dA, dB = _run_nano(p, n_nano, granule)
    _assert_ok(pu.compare(p, Y, dX, dA, dB), f"{dtype} N={n_nano} granule={granule}")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_accumulate_flag_adds_to_the_existing_gradients(dtype):
    from paper_2602_07263_amd import tlora
    p = wk.generate(wk.custom("acc", dtype, 128, 192, [4, 16, 9], [100, 0, 260], [2.0, 2.0, 0.5]), seed=8)
    Y, dX, dA, dB = _run_nano(p, 3, 32, flags=tlora.TLORA_BWD_ACCUMULATE, prefill=1.5)
    res = pu.compare(p, Y, dX, [a - 1.5 for a in dA], [b - 1.5 for b in dB])
    _assert_ok(res, f"accumulate/{dtype}")
    # the job without tokens keeps what was there
    assert np.all(dA[1] == 1.5) and np.all(dB[1] == 1.5)
    # and the plain call accumulates too
    import torch
    lp = tlora.LayerProblem.from_numpy(p)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dYt = torch.from_numpy(p.dY).to(device="cuda", dtype=tdt)
    Yt, dXt, dAt, dBt = lp.new_outputs()
    for t in dAt + dBt:
        t.fill_(-2.0)
    lp.fwd(Yt)
    lp.bwd(dYt, dXt, dAt, dBt, reuse_S=True, flags=tlora.TLORA_BWD_ACCUMULATE)
    torch.cuda.synchronize()
    res = pu.compare(p, Yt.float().cpu().numpy(), dXt.float().cpu().numpy(), [a.cpu().numpy() + 2.0 for a in dAt],
                     [b.cpu().numpy() + 2.0 for b in dBt])
    _assert_ok(res, f"accumulate plain/{dtype}")


# Nano-batches of which some run in the two-launch form of small batches and others in the general one: by their sizes, or by
# the ranks that are idle in them.  d_in d_out >= 2^19, so that dX runs against W as it lies in both.
MIXED = [
    # name, d_in, d_out, ranks, tokens, n_nano, granule, which nano-batches are small
    ("larger_last", 1024, 1024, [16], [700], 6, 100, [1, 1, 1, 1, 1, 0]),
    ("larger_in_between", 1024, 1024, [32, 30], [200, 250], 4, 75, [1, 0, 1, 0]),
    ("idle_ranks_later", 1024, 1024, [64, 16], [256, 256], 4, 128, [1, 1, 0, 0]),
    ("idle_ranks_first", 1024, 2048, [16, 64], [128, 256], 3, 128, [0, 1, 1]),
]


def small_nano_batches(prob, n_nano, granule):
    """Which nano-batches' backward runs in the two-launch form."""
    from paper_2602_07263_amd import tlora
    out = []
    for n in range(n_nano):
        _, _, off = tlora.tlora_nano_split(prob, n_nano, granule, n)
        sub, _keep = tlora.make_problem(tlora.TLORA_BF16, prob.d_in, prob.d_out, list(prob.ranks[:prob.num_jobs]), off,
                                        [1.0] * prob.num_jobs, 0x1000, 0x2000, [0x3000] * prob.num_jobs, [0x4000] * prob.num_jobs)
        c = tlora.tlora_plan_cuts(sub)
        out.append(int(c["bwd"] == (0, c["shrink_dy"])))
    return out


@pytest.mark.parametrize("case", MIXED, ids=[c[0] for c in MIXED])
def test_small_and_general_nano_batches_of_one_call(case):
    """dX of the general ones reads copies of the adapters that the small ones do without."""
    import torch
    from paper_2602_07263_amd import tlora
    name, d_in, d_out, ranks, tokens, n_nano, granule, small = case
    p = wk.generate(wk.custom(name, "bf16", d_in, d_out, ranks, tokens, [2.0] * len(ranks)), seed=12)
    lp = tlora.LayerProblem.from_numpy(p)
    assert small_nano_batches(lp.prob, n_nano, granule) == small
    lp._nano_ws(n_nano, granule)
    lp.ws.fill_(255)                                                    # (NaN in bf16 and fp32)
    dY = torch.from_numpy(p.dY).to(device="cuda", dtype=torch.bfloat16)
    Y, dX, dA, dB = lp.new_outputs()
    lp.fwd_nano(n_nano, granule, Y)
    lp.bwd_nano(n_nano, granule, dY, dX, dA, dB)
    torch.cuda.synchronize()
    n = lambda t: t.float().cpu().numpy()
    _assert_ok(pu.compare(p, n(Y), n(dX), [n(a) for a in dA], [n(b) for b in dB]), name)


def test_the_flag_after_small_nano_batches_makes_the_copy():
    """TLORA_BWD_REUSE_WT after a call that did without the copy of W^T: it is made where the first general nano-batch needs it,
    though the small ones before have no use for it, and found by the next call."""
    import torch
    from paper_2602_07263_amd import tlora
    for name, d_in, d_out, ranks, tokens, n_nano, granule, small in MIXED:
        p = wk.generate(wk.custom(name, "bf16", d_in, d_out, ranks, tokens, [2.0] * len(ranks)), seed=13)
        lp = tlora.LayerProblem.from_numpy(p)
        lp._nano_ws(n_nano, granule)
        lp.ws.fill_(255)
        dY = torch.from_numpy(p.dY).to(device="cuda", dtype=torch.bfloat16)
        first = None
        for flags in (0, tlora.TLORA_BWD_REUSE_WT, tlora.TLORA_BWD_REUSE_WT):
            Y, dX, dA, dB = lp.new_outputs()
            for t in (Y, dX, *dA, *dB):
                t.fill_(float("nan"))
            lp.fwd_nano(n_nano, granule, Y)
            lp.bwd_nano(n_nano, granule, dY, dX, dA, dB, flags)
            torch.cuda.synchronize()
            if first is None:
                first = [dX, *dA, *dB]
                n = lambda t: t.float().cpu().numpy()
                _assert_ok(pu.compare(p, n(Y), n(dX), [n(a) for a in dA], [n(b) for b in dB]), name)
            else:
                assert all(torch.equal(a, b) for a, b in zip(first, [dX, *dA, *dB])), (name, flags)


def test_reuse_of_the_transposed_weight():
    """A second backward with TLORA_BWD_REUSE_WT on the same workspace and W finds the copy."""
    import torch
    from paper_2602_07263_amd import tlora
    p = wk.generate(wk.custom("wt", "bf16", 256, 320, [8, 24], [200, 300]), seed=2)
    lp = tlora.LayerProblem.from_numpy(p)
    dY = torch.from_numpy(p.dY).to(device="cuda", dtype=torch.bfloat16)
    Y, dX, dA, dB = lp.new_outputs()
    lp.fwd(Y); lp.bwd(dY, dX, dA, dB, reuse_S=True)
    dX.fill_(float("nan"))
    lp.fwd(Y); lp.bwd(dY, dX, dA, dB, reuse_S=True, flags=tlora.TLORA_BWD_REUSE_WT)
    torch.cuda.synchronize()
    _assert_ok(pu.compare(p, Y.float().cpu().numpy(), dX.float().cpu().numpy(), [a.cpu().numpy() for a in dA],
                          [b.cpu().numpy() for b in dB]), "reuse Wt")


def test_transposed_weight_of_a_large_batch_serves_a_smaller_one():
    """The same jobs' next batch is smaller and takes the workspace, and W^T inside it, of the large one."""
    import torch
    from paper_2602_07263_amd import tlora
    large = wk.generate(wk.custom("wt_large", "bf16", 1024, 2048, [8, 24], [6000, 2192]), seed=3)
    small = wk.generate(wk.custom("wt_small", "bf16", 1024, 2048, [8, 24], [500, 401]), seed=4)
    lp = tlora.LayerProblem.from_numpy(large)
    lq = tlora.LayerProblem.from_numpy(small)
    lq = tlora.LayerProblem("bf16", 1024, 2048, small.ranks, small.offsets, small.scales, lq.X, lp.W, lp.A, lp.B)
    lq.ws, lq.ws_bytes = lp.ws, lp.ws_bytes
    up = lambda a: torch.from_numpy(a).to(device="cuda", dtype=torch.bfloat16)
    out = lp.new_outputs()
    lp.fwd(out[0]); lp.bwd(up(large.dY), *out[1:], reuse_S=True)
    Y, dX, dA, dB = lq.new_outputs()
    for t in (Y, dX, *dA, *dB):
        t.fill_(float("nan"))
    lq.fwd(Y); lq.bwd(up(small.dY), dX, dA, dB, reuse_S=True, flags=tlora.TLORA_BWD_REUSE_WT)
    torch.cuda.synchronize()
    small.W, small.A, small.B = large.W, large.A, large.B
    _assert_ok(pu.compare(small, Y.float().cpu().numpy(), dX.float().cpu().numpy(), [a.cpu().numpy() for a in dA],
                          [b.cpu().numpy() for b in dB]), "W^T of a larger batch")


def test_controller_in_the_loop():
    """Closed loop (Alg. 1, Phase 3): run a step with N nano-batches, feed a completion time to the controller, take
    its N for the next step.  The completion times that drive the controller are scripted (a fixed cost per
    nano-batch on top of a constant: what one GPU without communication to hide looks like), so the trajectory is
    the same on every machine; the steps themselves run on the GPU with each N the controller visits, and every one
    of them must stay correct.  Measured times are recorded but decide nothing."""
    import torch
    from oracle import aimd_oracle as aimd
    from paper_2602_07263_amd import tlora
    p = wk.generate(wk.custom("loop", "bf16", 512, 512, [8, 16, 32, 64], [1024, 512, 2048, 512]), seed=9)
    lp = tlora.LayerProblem.from_numpy(p)
    dY = torch.from_numpy(p.dY).to(device="cuda", dtype=torch.bfloat16)
    Y, dX, dA, dB = lp.new_outputs()
    c = tlora.tlora_aimd_init(32, n_max=64)
    scripted = lambda n: 1.0 + 0.05 * n
    visited, measured = [], []
    for step in range(12):
        n = c.n
        visited.append(n)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        lp.fwd_nano(n, 64, Y)
        lp.bwd_nano(n, 64, dY, dX, dA, dB)
        torch.cuda.synchronize()
        measured.append(time.perf_counter() - t0)
        tlora.tlora_aimd_update(c, scripted(n))
        _assert_ok(pu.compare(p, Y.float().cpu().numpy(), dX.float().cpu().numpy(), [a.cpu().numpy() for a in dA],
                              [b.cpu().numpy() for b in dB]), f"controller loop, N = {n}")
    print("N visited:", visited, "measured ms:", [round(t * 1e3, 3) for t in measured])
    # the same scripted times through the oracle's controller give the same trajectory
    n_ref, ref, prev = 32, [], None
    for step in range(12):
        ref.append(n_ref)
        t = scripted(n_ref)
        n_ref, prev = aimd.aimd_update(n_ref, t, prev, n_max=64), t
    assert visited == ref and min(visited) < 32, (visited, ref)

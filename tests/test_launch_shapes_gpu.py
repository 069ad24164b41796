"""Launches whose workgroups depend on the size: fp32 products in tiles of 32 (few tiles) and of 64, adapter packing in
tiles and pieces, chains of partial tiles, the optimizer's 16-byte path.  Sizes at the edges of each, against the fp64 oracle."""
import pytest

from paper_2602_07263_amd import workloads as wk
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

CASES = [
    # fp32: K-steps of 32 and remainders, tiles of 64 whose second half of 32 is empty, one-row and one-column units
    ("f32_one_step", "f32", 8, 8, [1], [1]),
    ("f32_edges", "f32", 40, 72, [1, 33, 5, 0], [1, 33, 64, 31]),
    ("f32_half_tiles", "f32", 96, 160, [32, 64], [97, 32]),
    ("f32_tiles_of_64", "f32", 264, 1032, [3, 65], [1000, 90]),          # 18 x 17 tiles forward, 18 x 5 backward
    # bf16: adapter tiles of 64 x 64 with one row or column over, pieces of 1024 chunks with one over, no chunk at all
    ("pack_one_rank", "bf16", 72, 8, [1], [3]),
    ("pack_over_the_edge", "bf16", 136, 1096, [65, 64, 0, 8, 129], [40, 1, 7, 0, 300]),
    # dA / dB in chunks of 256 tokens: chains of 1 to 16 partial tiles (added 8, 4, 2 and 1 at a time), blocks of one rank
    ("reduction_chains", "bf16", 64, 264, [8, 3, 33, 20, 1, 65, 16], [1, 257, 600, 1000, 1900, 2300, 3900]),
    ("pack_more_units_than_workgroups", "bf16", 1032, 520, [1] * 150 + [256], [2] * 151),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_sizes_at_the_edges_of_a_launch(case):
    name, dtype, d_in, d_out, ranks, tokens = case
    p = wk.generate(wk.custom(name, dtype, d_in, d_out, ranks, tokens, [2.0] * len(ranks)), seed=71)
    for reuse in (True, False):
        Y, dX, dA, dB, _ = pu.run_gpu(p, reuse_S=reuse)
        res = pu.compare(p, Y, dX, dA, dB)
        assert all(v <= 1.0 for v in res.values()), f"{name} reuse={reuse}: worst error / tolerance ratios {res}"


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shift", [0, 1, 2])
def test_optimizer_step_does_not_depend_on_alignment(dtype, shift):
    """Elementwise: one chunk of 4096 and a remainder, bases `shift` elements past a 64-element boundary -- within 1e-6 of
    the aligned state and the copy rounded from the call's own master."""
    import torch
    from paper_2602_07263_amd import tlora
    n = 4096 * 2 + 5
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(5)
    vals = [torch.randn(n, device="cuda", generator=g) for _ in range(3)] + [torch.rand(n, device="cuda", generator=g)]

    def step(at):
        bufs = [torch.zeros(n + 64, device="cuda") for _ in vals]
        views = [b[at:at + n].copy_(v) for b, v in zip(bufs, vals)]
        param = torch.zeros(n + 64, device="cuda", dtype=dt)[at:at + n]
        ws = torch.empty(tlora.tlora_adamw_workspace_bytes(1), dtype=torch.uint8, device="cuda")
        w, gr, m, v = views
        tlora.tlora_adamw_step([dict(param=param.data_ptr(), master=w.data_ptr(), grad=gr.data_ptr(), m=m.data_ptr(),
                                     v=v.data_ptr(), n=n, lr=1e-2, weight_decay=0.1, step=3)],
                               tlora.TLORA_BF16 if dtype == "bf16" else tlora.TLORA_F32, ws.data_ptr(), ws.numel(),
                               int(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        assert all(not b[:at].any() and not b[at + n:].any() for b in bufs)
        assert torch.equal(param, w.to(dt))
        return w, m, v

    for a, b in zip(step(0), step(shift)):
        assert torch.allclose(a, b, rtol=1e-6, atol=1e-7)


@pytest.mark.parametrize("d", [8, 2048, 2056, 4104, 8200])
def test_norm_rows_at_the_register_widths(d):
    """The norms hold rows of up to 2048, 4096 and 8192 features in registers and read wider ones twice."""
    from tests import test_mlp_gpu as tm
    tm.test_mlp_block_matches_oracle(("bf16", d, 64, [8, 3], [5, 2], [1.0, 2.0]))

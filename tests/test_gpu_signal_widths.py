"""The per-sequence signal kernels at both workgroup widths (1024 threads for up
to 256 sequences of 1024 tokens on average, the layer gap, or 1792, stability;
256 threads else) over lengths around their steps of four tokens a thread. Bars: J bit-exact, J_rand and RDA 1e-6, the gap's means 2e-7."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


LENGTHS = {"short": [0, 1, 2, 7, 255, 256, 257, 1100],
           "mid": [255, 511, 1023, 1024, 1025, 2047, 2049],  # 1024 to 1792 on average
           "long": [1023, 2049, 4095, 4097, 8191, 8192, 8193, 12289]}


@pytest.mark.parametrize("nb,kind", [(3, "short"), (512, "short"), (513, "short"), (40, "mid"), (5, "long"),
                                     (256, "mid"), (257, "mid"), (31, "long")])
def test_widths(nb, kind):
    import torch
    import paper_2608_29291_amd as ce
    from ce_workloads import build_layout
    from oracle import layer_gap as lg
    from test_gpu_stability import run_case
    rng = np.random.default_rng(nb)
    lens = [int(x) for x in rng.choice(LENGTHS[kind], size=nb)]
    lens[0], lens[1] = 4097, 5000
    segs = [[(n, 1), (2, 2)] for n in lens]
    mean = sum(lens) / nb + 2
    assert {"short": nb == 3 or mean < 1024, "mid": 1024 <= mean < 1792, "long": mean >= 1792}[kind]
    run_case(segs, 0.4, 0.6, 0.3, nb)
    offs, flags = build_layout(segs)
    T, d = len(flags), 64
    x = rng.standard_normal((T, d)).astype(np.float32)
    y = (x + rng.standard_normal((T, d))).astype(np.float32)
    pos = np.where(rng.random(T) < 0.5, np.arange(T), -1).astype(np.int32)
    up = lambda v: torch.from_numpy(np.ascontiguousarray(v)).cuda()
    batch = ce.Batch(up(offs), up(flags), None, 0.5, 0)
    cos = torch.empty(T, device="cuda")
    ra, rr, g = (torch.empty(nb, device="cuda") for _ in range(3))
    ce.ce_layer_gap(batch, up(x), up(y), up(pos), 0.004, cos, ra, rr, g)
    torch.cuda.synchronize()
    r_all, r_ret, gap, c = lg.redundancy_gap(x, y, offs, pos)
    np.testing.assert_allclose(ra.cpu().numpy(), r_all, rtol=0, atol=2e-7)
    np.testing.assert_allclose(rr.cpu().numpy(), r_ret, rtol=0, atol=2e-7)
    np.testing.assert_allclose(g.cpu().numpy(), gap, rtol=0, atol=3e-7)

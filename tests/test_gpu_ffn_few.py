"""FFN GEMMs of a few packed rows (a decode step: one always-kept token per
request) in the fused block against the oracle, at the edges of the row blocks
(16, 32, 64 rows, and 65 on the tiled kernels) and of the K split over a
workgroup's 8 waves. Bars as every block test: 2e-2 of max |Y|, 1e-2 of
max |FFN| beside one rounding of Y."""
import numpy as np
import pytest

from ce_workloads import TOK_GEN, TOK_KEEP, make_workload

pytestmark = pytest.mark.gpu
U, GN, K = 0, TOK_GEN, TOK_KEEP


def workload(n, n_sets, d, F):
    seqs = [[(1, K if n_sets == 1 or i % 3 else K | GN)] for i in range(n - 1)]
    seqs.append([(1, U), (3, GN if n_sets == 2 else U)])  # one retained row of four (keep 0.25)
    return make_workload("few", seqs, d=d, F=F, r_c=32, r_e=32, keep=0.25, dtype="bf16", seed=n, n_sets=n_sets,
                         biases=True)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 32, 33, 64, 65])
@pytest.mark.parametrize("n_sets", [1, 2])
@pytest.mark.parametrize("d,F", [(192, 320), (1088, 576)])  # 3, 5; 17, 9 lines of K; ragged over the 8 waves
def test_block(n, n_sets, d, F):
    import gpu_util as G
    wl = workload(n, n_sets, d, F)
    r = G.run_block(wl, inplace=bool(n & 1))
    assert int(r["koff"][-1]) == n
    err, _ = G.check_block(wl, r)
    print(f"[few n={n} sets={n_sets} d={d} F={F}] rel err {err:.2e}", flush=True)


@pytest.mark.parametrize("n", [1, 16, 33, 200, 300])
@pytest.mark.parametrize("n_sets", [1, 2])
@pytest.mark.parametrize("d,F", [(64, 128), (320, 576)])  # 2, 4; 10, 18 lines of K, ragged over the waves
def test_block_fp32(n, n_sets, d, F):
    """fp32 on row tiles of this kernel; 1e-5 of max |Y| and of max |FFN|."""
    import gpu_util as G
    a = n // 3 if n_sets == 2 else 0
    wl = make_workload("few32", [[(8, U), (max(n - a - 4, 0), K)], [(a, K | GN)]], d=d, F=F, r_c=32, r_e=32, keep=0.5,
                       dtype="f32", seed=n, n_sets=n_sets, biases=True)
    r = G.run_block(wl, inplace=bool(n & 1))
    err, _ = G.check_block(wl, r)
    print(f"[few fp32 n={n} sets={n_sets} d={d} F={F}] rel err {err:.2e}", flush=True)
    np.testing.assert_array_equal(r["y"], G.run_block(wl)["y"])


@pytest.mark.parametrize("n_sets", [1, 2])
@pytest.mark.parametrize("n", [3, 40])
def test_capacity_above_the_rows_and_determinism(n, n_sets):
    """A capacity above the packed count (more row blocks than rows)."""
    import torch
    import gpu_util as G
    import paper_2608_29291_amd as ce
    wl = workload(n, n_sets, 256, 512)
    outs = []
    for cap in (n, 60):
        dw = G.DevWorkload(wl, kept_capacity=cap)
        ki, ko = dw.new_idx()
        h = dw.hidden.clone()
        ce.ce_routed_block(dw.batch, h, h, dw.scorer, dw.ffn, dw.ws(ce.CE_WS_BLOCK), kept_idx_out=ki,
                           kept_offsets_out=ko)
        torch.cuda.synchronize()
        outs.append(G.host(h))
    ref = G.run_block(wl)
    G.check_block(wl, ref)
    np.testing.assert_array_equal(outs[0], ref["y"])
    # the blocks of 16 rows that hold rows are the same sums
    np.testing.assert_array_equal(outs[1], outs[0])


def test_staged_and_gap():
    """The staged calls and the fused layer gap on a decode step's rows."""
    import torch
    import oracle
    import gpu_util as G
    import paper_2608_29291_amd as ce
    from oracle import layer_gap
    wl = workload(21, 1, 448, 640)
    dw = G.DevWorkload(wl)
    f = torch.float32
    T, B = wl.T, wl.B
    cos, ra, rr, g = (torch.empty(k, dtype=f, device="cuda") for k in (T, B, B, B))
    ki, ko = dw.new_idx()
    out = torch.empty_like(dw.hidden)
    ce.ce_routed_block_gap(dw.batch, dw.hidden, out, dw.scorer, dw.ffn, dw.ws(ce.CE_WS_BLOCK_GAP), 0.004, cos, ra, rr,
                           g, kept_idx_out=ki, kept_offsets_out=ko)
    rows = dw.hidden[ki.long()].contiguous()
    ffn = torch.empty_like(rows)
    ce.ce_routed_ffn(dw.batch, rows, ki, ko, dw.ffn, ffn, dw.ws(ce.CE_WS_FFN))
    merged = torch.empty_like(dw.hidden)
    ce.ce_scatter_residual(dw.batch, ffn, ki, ko, dw.hidden, merged)
    torch.cuda.synchronize()
    y, kept = G.host(out), G.host(ki)
    # the staged path rounds the FFN once more before it adds the residual
    ref = oracle.routed_block(wl.hidden, wl.flags, wl.seq_offsets, wl.t, wl.keep, wl.scorer, wl.ffn,
                              kept_override=kept)
    assert G.ffn_term_err(y[kept], ref["y"][kept], wl.hidden[kept], "bf16") <= 1e-2
    assert G.ffn_term_err(G.host(merged)[kept], ref["y"][kept], wl.hidden[kept], "bf16") <= 1e-2
    pos = np.full(T, -1, np.int32)
    pos[kept] = np.arange(len(kept))
    _, _, gap, c = layer_gap.redundancy_gap(wl.hidden, y, wl.seq_offsets, pos)
    np.testing.assert_allclose(G.host(cos), c, rtol=0, atol=1e-7)
    np.testing.assert_allclose(G.host(g), gap, rtol=0, atol=3e-7)

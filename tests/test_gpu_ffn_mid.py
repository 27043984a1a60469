"""FFN GEMMs of mid-size packed counts (a request, a small batch) in the fused
block against the oracle, at the edges of the token tiles and of the pieces
over K, where the mid-size kernel takes one or both products. Bars as every
block test: 2e-2 of max |Y|, 1e-2 of max |FFN| beside one rounding of Y; the
layer gap's as in test_gpu_layer_gap.py. Widths with odd feature tiles (d =
576: 4.5 tiles of 128, F = 1088: 17 of 64) and enough K for several pieces.
These counts reach its tiles of 64 and 96 rows; test_gpu_ffn_routes.py has every
tile."""
import numpy as np
import pytest

from ce_workloads import TOK_GEN, TOK_KEEP, make_workload

pytestmark = pytest.mark.gpu
U, GN, K = 0, TOK_GEN, TOK_KEEP


def workload(n, n_sets, d, F):
    a = n // 3 if n_sets == 2 else 0  # generation rows: the second weight set
    segs = [[(8, U), (n - a - 4, K)], [(a, K | GN)]]  # 4 of 8 routable tokens stay
    return make_workload("mid", segs, d=d, F=F, r_c=32, r_e=32, keep=0.5, dtype="bf16", seed=n, n_sets=n_sets,
                         biases=True)


@pytest.mark.parametrize("n", [65, 96, 97, 159, 161, 257, 390])
@pytest.mark.parametrize("n_sets", [1, 2])
@pytest.mark.parametrize("d,F", [(576, 1088), (1536, 2304)])
def test_block_and_gap(n, n_sets, d, F):
    import torch
    import gpu_util as G
    import paper_2608_29291_amd as ce
    from oracle import layer_gap
    wl = workload(n, n_sets, d, F)
    r = G.run_block(wl, inplace=bool(n & 1))
    assert int(r["koff"][-1]) == n
    err, _ = G.check_block(wl, r)
    print(f"[mid n={n} sets={n_sets} d={d} F={F}] rel err {err:.2e}", flush=True)
    np.testing.assert_array_equal(r["y"], G.run_block(wl)["y"])  # in place or not, and again
    # the layer gap from the same launches, with a capacity above the rows
    dw = G.DevWorkload(wl, kept_capacity=n + 31)
    T, B = wl.T, wl.B
    cos, ra, rr, g = (torch.empty(k, device="cuda") for k in (T, B, B, B))
    out = torch.empty_like(dw.hidden)
    ki, ko = dw.new_idx()
    ce.ce_routed_block_gap(dw.batch, dw.hidden, out, dw.scorer, dw.ffn, dw.ws(ce.CE_WS_BLOCK_GAP), 0.004, cos, ra, rr,
                           g, kept_idx_out=ki, kept_offsets_out=ko)
    torch.cuda.synchronize()
    y, kept = G.host(out), G.host(ki)[:n]
    r2 = dict(r, y=y, kidx=G.host(ki))
    G.check_block(wl, r2)
    pos = np.full(T, -1, np.int32)
    pos[kept] = np.arange(n)
    _, _, gap, c = layer_gap.redundancy_gap(wl.hidden, y, wl.seq_offsets, pos)
    np.testing.assert_allclose(G.host(cos), c, rtol=0, atol=1e-7)
    np.testing.assert_allclose(G.host(g), gap, rtol=0, atol=3e-7)


@pytest.mark.parametrize("n_sets", [1, 2])
@pytest.mark.parametrize("n", [40, 300])  # the few-row kernel, this one
def test_staged_and_pruned(n, n_sets):
    """ce_routed_ffn and the staged calls on packed rows, and the pruned FFN
    with no sequence, some or all of them pruned against the staged masking on
    the same decisions: equal sums where nothing is pruned, else other orders
    of the same ones."""
    import torch
    import oracle
    import gpu_util as G
    import paper_2608_29291_amd as ce
    wl = workload(n, n_sets, 576, 1088)
    F = wl.d_ff
    dw = G.DevWorkload(wl)
    ki, ko = dw.new_idx()
    h = torch.empty_like(dw.hidden)
    ce.ce_routed_block(dw.batch, dw.hidden, h, dw.scorer, dw.ffn, dw.ws(ce.CE_WS_BLOCK), kept_idx_out=ki,
                       kept_offsets_out=ko)
    rows = dw.hidden[ki.long()].contiguous()
    whole, parts, pruned = (torch.empty_like(rows) for _ in range(3))
    act = torch.empty((len(rows), F), dtype=torch.bfloat16, device="cuda")
    wsf = dw.ws(ce.CE_WS_FFN)
    ce.ce_routed_ffn(dw.batch, rows, ki, ko, dw.ffn, whole, wsf)
    merged = torch.empty_like(dw.hidden)
    ce.ce_scatter_residual(dw.batch, whole, ki, ko, dw.hidden, merged)
    ce.ce_ffn_gateup(dw.batch, rows, ki, ko, dw.ffn, act, wsf)
    ce.ce_ffn_down(dw.batch, act, ki, ko, dw.ffn, parts, wsf)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(G.host(parts), G.host(whole))
    kept = G.host(ki)
    ref = oracle.routed_block(wl.hidden, wl.flags, wl.seq_offsets, wl.t, wl.keep, wl.scorer, wl.ffn,
                              kept_override=kept)
    assert G.ffn_term_err(G.host(merged)[kept], ref["y"][kept], wl.hidden[kept], "bf16") <= 1e-2
    norms = torch.empty(n_sets * F, device="cuda")
    ce.ce_ffn_down_colnorms(dw.ffn, norms)
    n_keep = 640
    mask = torch.zeros(F, dtype=torch.uint8, device="cuda")
    mask[n_keep:] = 1
    sal, lam = torch.empty((wl.B, F), device="cuda"), torch.empty(wl.B, device="cuda")
    use = torch.empty(wl.B, dtype=torch.uint8, device="cuda")
    wsp = dw.ws(ce.CE_WS_FFN_PRUNED)
    deltas = {"none": -1.0, "all": 1.0}
    for mode in ("none", "all", "some"):
        delta = deltas.get(mode)
        if delta is None:  # between the two sequences' leakages (one of them may have no rows)
            delta = float(G.host(lam).mean())
        ce.ce_routed_ffn_pruned(dw.batch, rows, ki, ko, dw.ffn, norms, n_keep, delta, pruned, sal, lam, use, wsp)
        ce.ce_ffn_gateup(dw.batch, rows, ki, ko, dw.ffn, act, wsf)
        act2 = act.clone()
        ce.ce_ffn_mask_channels(dw.batch, act, ko, mask, use)
        ce.ce_ffn_down(dw.batch, act, ki, ko, dw.ffn, parts, wsf)
        torch.cuda.synchronize()
        f, f2 = G.host(pruned), G.host(parts)
        # the segment sums: |z| of the staged activations, by hand
        if mode == "none":
            z = G.host(act2).astype(np.float64)
            off, fl = G.host(ko), wl.flags[kept]
            for b in range(wl.B):
                s = np.zeros(F)
                for j in range(off[b], off[b + 1]):
                    s += np.abs(z[j]) * G.host(norms)[(F if n_sets == 2 and fl[j] & 1 else 0):][:F]
                n_b = off[b + 1] - off[b]
                np.testing.assert_allclose(G.host(sal)[b], s / max(n_b, 1), rtol=1e-4, atol=1e-30)
        print(f"[mid pruned n={n} sets={n_sets} {mode}] pruned {int(use.sum())}/{wl.B}", flush=True)
        assert np.max(np.abs(f - f2)) <= 2.0 ** -7 * np.max(np.abs(f2))
        if mode == "none":
            np.testing.assert_array_equal(f, f2)

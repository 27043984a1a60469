"""The FFN GEMMs on every kernel and tile that the dispatch reaches, in the fused
block with its layer gap and in the pruned FFN, against float64 on the GPU. Each
case states the kernels it is for and asserts that the dispatch takes them, so a
change of the rules cannot empty it.

Bars, per element. Products of bf16 inputs are exact in fp32 and summed over K
values: sum |a w| sqrt(K) 2^-24, and 2^-8 of the result for its rounding to
bf16. The activation's errors pass through SwiGLU with its derivatives (|silu'|
<= 1.1) and through the down product with its weights' magnitudes; the output
adds one rounding. The layer gap's bars as in test_gpu_layer_gap.py.
"""
import pytest

TILES, WIDE, FEW, MID = range(4)
N_KEEP = 0.75  # share of the channels that the pruned FFN keeps

# (d, d_ff, packed rows, weight sets): (gate/up kernel, down kernel)
CASES = {
    # mid-size kernel: its token tiles of 64 to 256 rows with 128 and 256 weight
    # rows, at the counts where one tile hands over to the next (multiples of its
    # rows, and one more)
    **{(1024, 4096, n, s): (MID, MID) for n in (65, 96, 256, 257, 384, 385, 512, 513, 640, 641, 768, 769, 1024, 1025)
       for s in (1, 2) if (n, s) not in ((1024, 2),)},
    (576, 1088, 3600, 1): (MID, MID), (576, 1088, 3500, 2): (MID, MID),
    (1024, 4096, 3400, 1): (WIDE, MID), (1536, 2304, 1441, 2): (MID, MID),
    (1536, 8960, 97, 1): (MID, MID), (1536, 8960, 193, 1): (MID, MID), (1536, 8960, 289, 1): (MID, MID),
    (1536, 8960, 402, 1): (MID, MID), (1536, 8960, 673, 1): (WIDE, MID), (1536, 8960, 864, 2): (MID, MID),
    (1536, 8960, 2400, 1): (WIDE, MID), (1536, 8960, 2688, 1): (WIDE, MID),
    # 256 x 256 kernel: absorbed last tiles (1 and 32 rows), split gate/up (2 to 5
    # pieces), split down (2 to 11), whole tiles
    (1536, 8960, 513, 1): (WIDE, MID), (1536, 8960, 544, 1): (WIDE, MID), (1536, 8960, 545, 1): (WIDE, MID),
    (1536, 8960, 2689, 1): (WIDE, WIDE), (1536, 8960, 3329, 1): (WIDE, WIDE), (1536, 8960, 3300, 2): (WIDE, WIDE),
    (1024, 4096, 2600, 1): (WIDE, MID), (2048, 11008, 1400, 1): (WIDE, MID), (2048, 11008, 2100, 1): (WIDE, WIDE),
    (3584, 18944, 490, 1): (WIDE, MID), (3584, 18944, 800, 1): (WIDE, WIDE), (3584, 18944, 500, 2): (WIDE, WIDE),
    (3584, 18944, 3600, 1): (WIDE, WIDE), (3584, 18944, 4615, 1): (WIDE, WIDE),
    # down on the smaller tiles where few 256 x 256 ones cannot split
    (2048, 11008, 4200, 1): (WIDE, TILES), (3584, 18944, 2400, 1): (WIDE, TILES),
    # few-row kernel, one row block to four, and past it
    (1024, 4096, 16, 1): (FEW, FEW), (1024, 4096, 17, 2): (FEW, FEW), (1024, 4096, 33, 1): (FEW, FEW),
    (1024, 4096, 64, 2): (FEW, FEW),
}


def test_cases_take_the_kernels_they_name():
    """And together every tile of the mid-size kernel and every kind of split."""
    G = pytest.importorskip("gpu_util")
    seen = [set(), set()]
    for (d, F, n, s), kernels in CASES.items():
        for mode in (0, 1):
            r = G.ffn_route(mode, n, d, F, s)
            assert r[0] == kernels[mode], (d, F, n, s, mode, r)
            seen[mode].add(r[:3] if r[0] == MID else (r[0], min(r[3], 5), r[4]))
    assert {x[1:] for x in seen[0] if x[0] == MID} == {(2, m) for m in (2, 3, 4, 5, 6, 8)} | {(4, m) for m in (3, 4, 5)}
    assert {x[1:] for x in seen[1] if x[0] == MID} == {(2, m) for m in (2, 3, 4, 5, 6, 8)}
    assert {x for x in seen[0] if x[0] == WIDE} >= {(WIDE, 1, 1), (WIDE, 2, 0), (WIDE, 4, 0), (WIDE, 5, 0)}
    assert {x for x in seen[1] if x[0] == WIDE} >= {(WIDE, p, 0) for p in (1, 2, 3, 4, 5)}


def ffn64(torch, x, wg, wu, wd):
    """float64 SwiGLU of bf16 rows, with the bound on |z_gpu - z|."""
    g, u = x.double() @ wg.double().T, x.double() @ wu.double().T
    e = x.shape[1] ** 0.5 * 2.0 ** -24
    eg, eu = (e * (x.abs().float() @ w.abs().float().T).double() for w in (wg, wu))
    s = g * torch.sigmoid(g)
    z = s * u
    return z, 1.1 * u.abs() * eg + s.abs() * eu + (2.0 ** -8 + 2.0 ** -20) * z.abs()


def down64(torch, z, ez, wd):
    """float64 down product, with the bound on the GPU's before its rounding."""
    w = wd.double()
    y = z @ w.T
    return y, (ez + z.shape[1] ** 0.5 * 2.0 ** -24 * z.abs()) @ w.abs().T


# two sequences each, and a few with so many that a token tile holds more of them
# than its segment sums (9 rows each, and 60)
BATCHES = [(*c, 2) for c in CASES] + [(1536, 8960, 2700, 1, 300), (1536, 8960, 3420, 1, 57), (1536, 8960, 3420, 2, 57),
                                      (1024, 4096, 900, 1, 100), (1024, 4096, 48, 1, 24)]


@pytest.mark.gpu
@pytest.mark.parametrize("d,F,n,sets,B", BATCHES)
def test_block_gap_and_pruned(d, F, n, sets, B):
    import torch

    import gpu_util as G
    import paper_2608_29291_amd as ce
    g = torch.Generator("cuda").manual_seed(n + sets)
    bf = torch.bfloat16

    def rnd(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    # kept tokens and a few routable ones in each sequence, of which half stay
    lens = [n // 3, n - n // 3] if B == 2 else [n // B] * B
    extra = min(8, 2 * min(lens))
    flags, offs = [], [0]
    for k in lens:
        f = torch.full((k - extra // 2 + extra,), ce.CE_TOK_KEEP, dtype=torch.uint8)
        f[torch.randperm(len(f), generator=torch.Generator().manual_seed(k))[:extra]] = 0
        if sets == 2:
            f[1::3] |= ce.CE_TOK_GEN
        flags.append(f)
        offs.append(offs[-1] + len(f))
    flags = torch.cat(flags).cuda()
    T = offs[-1]
    batch = ce.Batch(torch.tensor(offs, dtype=torch.int32).cuda(), flags, torch.full((B,), 0.5, device="cuda"), 0.5, n)
    sc = ce.Scorer(rnd(32, d).to(bf), rnd(32), rnd(4, 32, d).to(bf), rnd(4, 32))
    W = [((rnd(F, d) * d ** -0.5).to(bf), (rnd(F, d) * d ** -0.5).to(bf), (rnd(d, F) * F ** -0.5).to(bf))
         for _ in range(sets)]
    ffn = ce.FFN(*[list(x) for x in zip(*W)])
    h = rnd(T, d).to(bf)
    out = torch.full_like(h, 3.0)
    ki, ko = torch.full((n,), -7, dtype=torch.int32, device="cuda"), torch.empty(B + 1, dtype=torch.int32, device="cuda")
    cos, (ra, rr, gap) = torch.empty(T, device="cuda"), (torch.empty(B, device="cuda") for _ in range(3))
    ws = ce.alloc_workspace(ce.CE_WS_BLOCK_GAP, batch, d, F, ce.CE_BF16)
    ce.ce_routed_block_gap(batch, h, out, sc, ffn, ws, 0.004, cos, ra, rr, gap, kept_idx_out=ki, kept_offsets_out=ko)
    plain = h.clone()
    ce.ce_routed_block(batch, plain, plain, sc, ffn, ce.alloc_workspace(ce.CE_WS_BLOCK, batch, d, F, ce.CE_BF16))
    torch.cuda.synchronize()
    assert ko.tolist() == [sum(lens[:b]) for b in range(B + 1)]
    kept = ki.long()
    dropped = torch.ones(T, dtype=torch.bool, device="cuda")
    dropped[kept] = False
    assert torch.equal(out[dropped], h[dropped]) and torch.equal(out, plain)

    # the pruned FFN on the packed rows: no sequence pruned, all, and half of them
    rows = h[kept].contiguous()
    norms = torch.empty(sets * F, device="cuda")
    ce.ce_ffn_down_colnorms(ffn, norms)
    n_keep = int(N_KEEP * F) // 64 * 64
    sal, lam = torch.empty((B, F), device="cuda"), torch.empty(B, device="cuda")
    use = torch.empty(B, dtype=torch.uint8, device="cuda")
    wsp = ce.alloc_workspace(ce.CE_WS_FFN_PRUNED, batch, d, F, ce.CE_BF16)
    full, cut, some = (torch.full_like(rows, float("nan")) for _ in range(3))
    for delta, y in ((-1.0, full), (1.0, cut), (None, some)):
        delta = float(lam.mean()) if delta is None else delta
        ce.ce_routed_ffn_pruned(batch, rows, ki, ko, ffn, norms, n_keep, delta, y, sal, lam, use, wsp)
        torch.cuda.synchronize()
        assert torch.equal(use.bool(), lam <= delta)
    assert 0 < int(use.sum()) < B
    # an empty kept prefix, and one of all channels; the staged calls, each of
    # which clears its own counters, and the whole call twice on one workspace
    edge, ident = (torch.full_like(rows, float("nan")) for _ in range(2))
    ce.ce_routed_ffn_pruned(batch, rows, ki, ko, ffn, norms, 0, 1.0, edge, torch.empty_like(sal), torch.empty_like(lam),
                            torch.empty_like(use), wsp)
    ce.ce_routed_ffn_pruned(batch, rows, ki, ko, ffn, norms, F, 1.0, ident, torch.empty_like(sal), torch.empty_like(lam),
                            torch.empty_like(use), wsp)
    wsf = ce.alloc_workspace(ce.CE_WS_FFN, batch, d, F, ce.CE_BF16)
    once, again, staged = (torch.full_like(rows, float("nan")) for _ in range(3))
    act = torch.full((n, F), float("nan"), dtype=bf, device="cuda")
    ce.ce_routed_ffn(batch, rows, ki, ko, ffn, once, wsf)
    ce.ce_routed_ffn(batch, rows, ki, ko, ffn, again, wsf)
    ce.ce_ffn_gateup(batch, rows, ki, ko, ffn, act, wsf)
    ce.ce_ffn_down(batch, act, ki, ko, ffn, staged, wsf)
    torch.cuda.synchronize()
    assert not edge.any() and torch.equal(ident, full)
    assert torch.equal(once, again) and torch.equal(once, staged)
    seq = torch.repeat_interleave(torch.arange(B, device="cuda"), torch.tensor(lens, device="cuda"))

    sets_of = (flags[kept] & ce.CE_TOK_GEN != 0).long() if sets == 2 else torch.zeros(n, dtype=torch.long, device="cuda")
    sal64, esal = torch.zeros((B, F), dtype=torch.float64, device="cuda"), torch.zeros((B, F), dtype=torch.float64, device="cuda")
    worst = 0.0
    for s in range(sets):
        mine = (sets_of == s).nonzero()[:, 0]
        for at in mine.split(512):
            z, ez = ffn64(torch, rows[at], *W[s])
            cuts = use[seq[at]].bool()
            for y, k, m in ((full, F, None), (once, F, None), (cut, n_keep, None), (some, F, ~cuts), (some, n_keep, cuts)):
                ref, err = down64(torch, z[:, :k], ez[:, :k], W[s][2][:, :k])
                over = (y[at].double() - ref).abs() / (err + 2.0 ** -8 * ref.abs())
                over = over if m is None else over[m]
                assert over.numel() == 0 or over.max() <= 1, (k, over.max())
            ref, err = down64(torch, z, ez, W[s][2])
            ref += rows[at].double()
            over = (out[kept[at]].double() - ref).abs() / (err + 2.0 ** -8 * ref.abs())
            worst = max(worst, float(over.max()))
            nm = norms[s * F:(s + 1) * F].double()
            share = nm / torch.tensor(lens, device="cuda")[seq[at], None]
            sal64.index_add_(0, seq[at], z.abs() * share)
            esal.index_add_(0, seq[at], ez * share)
    print(f"[ffn {d}/{F} n={n} sets={sets} B={B}] {[G.ffn_route(m, n, d, F, sets)[:4] for m in (0, 1)]} block {worst:.2f} of the bar",
          flush=True)
    assert worst <= 1
    assert ((sal.double() - sal64).abs() <= esal + 2.0 ** -16 * sal64).all()
    # the layer gap's cosines, of the states as stored
    x, y = h.double(), out.double()
    c = (x * y).sum(1) / (x.norm(dim=1) * y.norm(dim=1))
    assert (cos.double() - c).abs().max() <= 1e-7


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1024, 1025])
def test_fp32_handover(n):
    """fp32 down: the K-split kernel up to 1024 rows, 32 x 32 tiles past it, each
    with its own slots of the layer gap's sums."""
    import numpy as np
    import torch

    import gpu_util as G
    import paper_2608_29291_amd as ce
    from oracle import layer_gap
    from ce_workloads import TOK_KEEP, make_workload
    assert [G.ffn_route(1, n, 256, 512, dtype="f32")[0], G.ffn_route(0, n, 256, 512, dtype="f32")[0]] == \
        [FEW if n <= 1024 else TILES, FEW]
    wl = make_workload("few32", [[(8, 0), (n - 4, TOK_KEEP)]], d=256, F=512, r_c=32, r_e=32, keep=0.5, dtype="f32",
                       seed=n, biases=True)
    r = G.run_block(wl)
    assert int(r["koff"][-1]) == n
    err, _ = G.check_block(wl, r)
    print(f"[fp32 n={n}] rel err {err:.2e}", flush=True)
    dw = G.DevWorkload(wl)
    T, B = wl.T, wl.B
    cos, ra, rr, gap = (torch.empty(k, device="cuda") for k in (T, B, B, B))
    out, (ki, ko) = torch.empty_like(dw.hidden), dw.new_idx()
    ce.ce_routed_block_gap(dw.batch, dw.hidden, out, dw.scorer, dw.ffn, dw.ws(ce.CE_WS_BLOCK_GAP), 0.004, cos, ra, rr,
                           gap, kept_idx_out=ki, kept_offsets_out=ko)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(G.host(out), r["y"])
    pos = np.full(T, -1, np.int32)
    pos[G.host(ki)] = np.arange(n)
    _, _, want, c = layer_gap.redundancy_gap(wl.hidden, G.host(out), wl.seq_offsets, pos)
    np.testing.assert_allclose(G.host(cos), c, rtol=0, atol=1e-7)
    np.testing.assert_allclose(G.host(gap), want, rtol=0, atol=3e-7)

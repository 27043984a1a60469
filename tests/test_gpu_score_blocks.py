"""The single-launch scorer at every number of 32-rank blocks it has a variant
for (1 to 16 with 32-token tiles, 1 to 12 with 128-token tiles, core and
expansion split in several ways), fp32 and bf16, K of one to ten slabs, against
float64.

Bar: fp32 products of bf16 or fp32 inputs, summed in fp32 over d <= 320 values
and 512 ranks: each logit is off by at most about sqrt(d + r) 2^-24 of the sum
of its terms' magnitudes; 1e-5 of the largest logit leaves a factor of ten.
"""
import pytest

pytestmark = pytest.mark.gpu


def reference(torch, h, flags, m, sc, ce):
    def mlp(x, w1, b1, w2, b2):
        a = x @ w1.double().T + b1.double()
        return (a * torch.sigmoid(a)) @ w2.double() + b2
    x = h.double()
    out = mlp(x, sc.w1_core, sc.b1_core, sc.w2_core, float(sc.b2_core))
    gen = (flags & ce.CE_TOK_GEN) != 0
    if gen.any() and sc.w1_exp is not None:
        out[gen] += mlp(x[gen], sc.w1_exp[m], sc.b1_exp[m], sc.w2_exp[m], float(sc.b2_exp[m]))
    out[(flags & ce.CE_TOK_KEEP) != 0] = float("inf")
    return out


def check(T, und, core, exp, dtype, slabs):
    """T tokens, `und` for understanding, then generation with four kept ones."""
    import torch

    import paper_2608_29291_amd as ce
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    d = 64 * slabs  # bf16 values of a slab; fp32 takes two slabs for them
    g = torch.Generator("cuda").manual_seed(100 * core + exp + d)

    def rnd(*shape, to=torch.float32):
        return (torch.randn(shape, generator=g, device="cuda") * shape[-1] ** -0.5).to(to)

    r_c, r_e = 32 * core, 32 * exp
    sc = ce.Scorer(rnd(r_c, d, to=dt), rnd(r_c), rnd(4, r_e, d, to=dt), rnd(4, r_e), b1_core=rnd(r_c), b2_core=0.25,
                   b1_exp=rnd(4, r_e), b2_exp=rnd(4))
    flags = torch.zeros(T, dtype=torch.uint8)
    flags[und:] = ce.CE_TOK_GEN
    flags[und + 10:und + 14] = ce.CE_TOK_KEEP
    flags = flags.cuda()
    h = torch.randn((T, d), generator=g, device="cuda").to(dt)
    batch = ce.Batch(torch.tensor([0, T], dtype=torch.int32).cuda(), flags, torch.tensor([0.6]).cuda(), 0.5, T)
    logits = torch.empty(T, device="cuda")
    ce.ce_score(batch, h, sc, logits)
    torch.cuda.synchronize()
    ref = reference(torch, h, flags, 2, sc, ce)
    fin = torch.isfinite(ref)
    assert torch.equal(torch.isfinite(logits), fin)
    err = ((logits.double() - ref)[fin].abs().max() / ref[fin].abs().max()).item()
    print(f"[score blocks T={T} {core}+{exp} {dtype} slabs={slabs}] err {err:.1e}", flush=True)
    assert err <= 1e-5


@pytest.mark.parametrize("slabs", [1, 2, 3, 5])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("core,exp", [(1, 1), (2, 1), (3, 2), (4, 4), (6, 1), (8, 3), (9, 1), (9, 4), (12, 2), (15, 1)])
def test_rank_blocks(core, exp, dtype, slabs):
    check(77, 40, core, exp, dtype, slabs)  # an understanding tile (core blocks only), a mixed one, a ragged one


@pytest.mark.parametrize("slabs", [1, 2, 3, 5])
@pytest.mark.parametrize("core,exp", [(n, 1) for n in range(1, 12)] + [(4, 8), (8, 4)])
def test_rank_blocks_of_large_tiles(core, exp, slabs):
    """128-token tiles: `core` blocks up to the mixed tile, core + exp after it."""
    T = 16500  # 516 tiles of 32 tokens are three rounds of the 256 CUs, 129 of 128 are one: always the larger
    rounds = [-(-T // t // 256) * (t + 32 * (core + exp)) for t in (32, 128)]
    assert rounds[1] < rounds[0]
    check(T, 6000, core, exp, "bf16", slabs)

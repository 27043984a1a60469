"""The 128-query attention kernel where its pipeline fills and drains (one, two
and three key tiles, each with a part of a block of 32 keys), where the walk to
a workgroup's sequence changes (64 sequences), and next to rows that belong to
nobody's softmax: keys and values past a sequence's end are fetched with its
last tile and must not reach its output.

Bar: max |O_gpu - O_ref| <= 2^-8 max|v| + 1e-6 (probabilities and outputs each
rounded to bf16, 2^-9 of a convex combination of value rows apiece).
"""
import numpy as np
import pytest

from ce_workloads import make_attention_inputs
from oracle import attention as oa

pytestmark = pytest.mark.gpu

DH = 128


def run(q, k, v, qo, ko, causal):
    import torch

    import gpu_util as G
    import paper_2608_29291_amd as ce
    dq, dk, dv = (G.to_dev(x, torch.bfloat16) for x in (q, k, v))
    o = torch.full(dq.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    ce.ce_routed_attention(dq, dk, dv, o, G.to_dev(qo), G.to_dev(ko), causal, DH ** -0.5)
    torch.cuda.synchronize()
    return G.host(o)


def check(got, ref, v):
    assert float(np.max(np.abs(got - ref))) <= 2.0 ** -8 * float(np.max(np.abs(v))) + 1e-6


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 161, 192, 193])
def test_tile_edges(n, causal):
    q_lens, kv_lens = [n, 130, 40], [n, n, 200 + n]
    q, k, v, qo, ko = make_attention_inputs(q_lens, kv_lens, 4, 2, DH, seed=n + causal)
    check(run(q, k, v, qo, ko, causal), oa.attention(q, k, v, qo, ko, 2, causal, DH ** -0.5), v)


@pytest.mark.parametrize("B", [1, 63, 64, 65])
def test_sequence_walk(B):
    rng = np.random.default_rng(B)
    lens = [int(x) for x in rng.integers(0, 90, size=B)]
    lens[0] = 0
    lens[-1] = 300  # several query tiles in the last sequence
    q, k, v, qo, ko = make_attention_inputs(lens, lens, 2, 1, DH, seed=B)
    check(run(q, k, v, qo, ko, True), oa.attention(q, k, v, qo, ko, 1, True, DH ** -0.5), v)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("n", [33, 65, 100, 160])
def test_neighbours_do_not_leak(n, bad):
    """The sequence after holds NaN or infinity in every key and value."""
    lens = [n, 64]
    q, k, v, qo, ko = make_attention_inputs(lens, lens, 2, 1, DH, seed=n)
    ref = oa.attention(q, k, v, qo, ko, 1, False, DH ** -0.5)
    k[n:], v[n:] = bad, bad
    got = run(q, k, v, qo, ko, False)
    check(got[:n], ref[:n], v[:n])

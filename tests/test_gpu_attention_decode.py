"""Routed attention with few queries per sequence (decode and speculative
steps over the compressed cache) against the float64 oracle, at the sizes where
the key chunks, the 32-key tiles and the 32 (query, head) rows of a work item
end. Tolerance as in test_gpu_attention.py: the probabilities' and the output's
bf16 roundings, 2^-8 max|v|; adding the chunks' fp32 results changes neither.
"""
import numpy as np
import pytest

from ce_workloads import make_attention_inputs
from oracle import attention as oa

pytestmark = pytest.mark.gpu
DH = 128


def run(q, k, v, qo, ko, causal, ws=True):
    import ctypes
    import torch
    import gpu_util as G
    import paper_2608_29291_amd as ce
    bf = torch.bfloat16
    dq, dk, dv, dqo, dko = G.to_dev(q, bf), G.to_dev(k, bf), G.to_dev(v, bf), G.to_dev(qo), G.to_dev(ko)
    o = torch.full(dq.shape, float("nan"), dtype=bf, device="cuda")
    if ws:
        ce.ce_routed_attention(dq, dk, dv, o, dqo, dko, causal, DH ** -0.5)
    else:  # the C entry point without a workspace: no sequence is cut
        at = ce.CEAttn(len(qo) - 1, q.shape[1], k.shape[1], DH, dqo.data_ptr(), dko.data_ptr(), len(q), len(k),
                       int(causal), DH ** -0.5, ce.CE_BF16)
        st = ce.lib.ce_routed_attention(ctypes.byref(at), dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), o.data_ptr(),
                                        torch.cuda.current_stream().cuda_stream)
        assert st == ce.CE_OK
    torch.cuda.synchronize()
    return G.host(o)


CASES = {
    # one query: cache ends at the edges of tiles and chunks
    "edges": ([1] * 9, [1, 31, 32, 33, 127, 128, 129, 256, 1000], 12, 2),
    "long": ([1, 1], [5003, 40], 28, 4),
    "ungrouped": ([1, 1, 1], [700, 300, 129], 4, 4),
    "wide_group": ([1, 1], [900, 257], 32, 1),  # all 32 rows of an item
    # several queries: 4 x 7 rows fit an item, 5 x 7 need two (that sequence is not cut)
    "speculative": ([4, 1, 5, 2, 0, 1, 3, 1], [900, 1300, 700, 2, 400, 0, 333, 650], 28, 4),
    # all queries in one sequence of many; more queries than keys
    "skewed": ([40] + [0] * 7 + [1] * 40, [600] + [9] * 7 + [35] * 40, 12, 2),
    "short_cache": ([3, 2], [1, 2], 12, 2),
    # mixed batches: a prefill among decode steps and empty sequences; sequences
    # of 2 to 7 tiles of rows over long caches (tiles times chunks); around the
    # line to 128-query tiles (32 queries), cut and not, one row per query and odd
    "prefill": ([260] + [1] * 30 + [0] * 35, [260] + [700] * 30 + [5] * 35, 28, 4),
    "tiles": ([5, 1, 15, 31] + [0] * 8, [3000, 900, 1500, 4001] + [0] * 8, 28, 4),
    "line": ([31, 32, 33] + [0] * 20, [700, 699, 701] + [3] * 20, 28, 4),
    "line_cut": ([33, 32] + [0] * 13, [4001, 2500] + [3] * 13, 12, 2),
    "ungrouped_line": ([40, 33, 1], [2000, 100, 200], 4, 4),
    "odd_group": ([129, 2] + [0] * 20, [200, 3000] + [0] * 20, 20, 4),
    # many sequences that are cut: two chunks of 128 keys and a bit, three, one
    "cut": ([1] * 40, [129, 128, 257, 130] * 10, 28, 4),
    # the same at chunks of 128 keys (256 where caches are that short on average),
    # and the line below which nothing is cut
    "edges_128": ([1] * 9, [1, 128, 129, 255, 256, 257, 384, 385, 1500], 12, 2),
    "cut_128": ([1] * 41, [129, 128, 257, 130] * 10 + [6000], 28, 4),
    "one_whole": ([1], [384], 12, 2),
    "one_cut": ([1], [385], 12, 2),
    "many": ([1] * 600, [(7 * i) % 90 for i in range(600)], 4, 2),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("causal", [False, True])
def test_few_queries(name, causal):
    ql, kl, h, hkv = CASES[name]
    assert sum(ql) * (h // hkv) <= 32 * len(ql)  # the shape of call that takes this kernel
    q, k, v, qo, ko = make_attention_inputs(ql, kl, h, hkv, DH, seed=len(name))
    ref = oa.attention(q, k, v, qo, ko, hkv, causal, DH ** -0.5)
    tol = 2.0 ** -8 * float(np.max(np.abs(v))) + 1e-6
    for ws in (True, False):
        got = run(q, k, v, qo, ko, causal, ws)
        err = float(np.max(np.abs(got - ref)))
        print(f"[decode {name} causal={causal} ws={ws}] max err {err:.3e} (bar {tol:.3e})", flush=True)
        assert err <= tol
        np.testing.assert_array_equal(got, run(q, k, v, qo, ko, causal, ws))


@pytest.mark.parametrize("kind", ["query", "key prefix", "one key", "score", "value", "infinite value"])
@pytest.mark.parametrize("causal", [False, True])
def test_not_finite(kind, causal):
    """NaN and infinity come out of the rows and heads that see them, and of no
    others, whether a cache is cut into chunks (of 128 keys here) or not."""
    h, hkv = 4, 2
    q, k, v, qo, ko = make_attention_inputs([1, 1], [1805, 300], h, hkv, DH, seed=5)
    if kind == "query":
        q[0, 1, 7] = q[1, 0, 3] = np.nan
        want = [((0, 1), np.nan), ((1, 0), np.nan)]
    elif kind == "key prefix":  # the first ten chunks of one cache, all of the other
        k[:1400] = k[1805:] = np.nan
        want = [(..., np.nan)]
    elif kind == "one key":
        k[1700, 0, 5] = np.nan
        want = [((0, slice(0, 2)), np.nan)]
    elif kind == "score":  # 1e40: infinite in fp32, inf - inf
        q[0, 2, 5] = k[900, 1, 5] = 1e20
        q[0, 3, 5] = 0
        want = [((0, 2), np.nan)]
    elif kind == "value":
        v[1100, 0, 64] = np.nan
        want = [((0, slice(0, 2), 64), np.nan)]
    else:  # in the last chunk, the fifteenth
        v[1800, 1, 9] = np.inf
        want = [((0, slice(2, 4), 9), np.inf)]
    with np.errstate(all="ignore"):
        ref = oa.attention(q, k, np.where(np.isfinite(v), v, 0), qo, ko, hkv, causal, DH ** -0.5)
    for at, x in want:
        ref[at] = x
    tol = 2.0 ** -8 * float(np.max(np.abs(v[np.isfinite(v)]))) + 1e-6
    for ws in (True, False):
        got = run(q, k, v, qo, ko, causal, ws)
        print(f"[decode {kind} causal={causal} ws={ws}] {np.isnan(got).sum()} NaN, {np.isinf(got).sum()} inf", flush=True)
        np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
        np.testing.assert_array_equal(np.isinf(got), np.isinf(ref))
        fin = np.isfinite(ref)
        assert np.max(np.abs(got[fin] - ref[fin]), initial=0) <= tol


def test_own_stream_and_capture():
    """On another stream, and captured with replays between eager calls."""
    import torch
    import gpu_util as G
    import paper_2608_29291_amd as ce
    ql, kl, h, hkv = CASES["long"]
    q, k, v, qo, ko = make_attention_inputs(ql, kl, h, hkv, DH, seed=3)
    want = run(q, k, v, qo, ko, True)
    bf = torch.bfloat16
    args = [G.to_dev(q, bf), G.to_dev(k, bf), G.to_dev(v, bf)]
    o, dqo, dko = torch.zeros_like(args[0]), G.to_dev(qo), G.to_dev(ko)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    ce.ce_routed_attention(*args, o, dqo, dko, True, DH ** -0.5, stream=side)
    side.synchronize()
    np.testing.assert_array_equal(G.host(o), want)
    # a stream that is only its raw handle, as another library's wrapper has it
    import types
    o.zero_()
    side.wait_stream(torch.cuda.current_stream())
    ce.ce_routed_attention(*args, o, dqo, dko, True, DH ** -0.5, stream=types.SimpleNamespace(cuda_stream=side.cuda_stream))
    side.synchronize()
    np.testing.assert_array_equal(G.host(o), want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ce.ce_routed_attention(*args, o, dqo, dko, True, DH ** -0.5)
    for _ in range(3):
        o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(G.host(o), want)
        run(q, k, v, qo, ko, False)

"""The Python entry points' native part: results made by the call, results passed in, refused arguments."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("sizes,max_path", [([1], 1), ([0, 5, 0], 3), ([70, 8, 33], 9), ([130], 200)])
def test_paths_made_by_the_call_end_in_minus_one(sizes, max_path):
    import torch
    from paper_2510_26577_amd import verify, workloads as wl
    rng = np.random.default_rng(5)
    trees = [wl.tree_uniform(rng, t, 8) for t in sizes if t]
    cu_T = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    tok = rng.integers(0, 3, cu_T[-1]).astype(np.int32)
    want = rng.integers(0, 3, cu_T[-1]).astype(np.int32)
    args = (d(np.concatenate(trees).astype(np.int32)), d(cu_T), d(tok), d(want), max_path)
    given = torch.full((len(sizes), max_path), -7, dtype=torch.int32, device="cuda")
    p0, n0, t0 = verify.accept_greedy(*args, path=given)
    p1, n1, t1 = verify.accept_greedy(*args)
    assert p0 is given and torch.equal(n0, n1) and torch.equal(t0, t1)
    past = torch.arange(max_path, device="cuda")[None, :] >= n1[:, None]
    assert torch.equal(p1, torch.where(past, torch.full_like(p1, -1), p0)) and bool((p0[past] == -7).all())


def test_results_and_scratch_passed_in_are_used_and_refusals_raise():
    import torch
    from paper_2510_26577_amd import binding, workloads as wl
    from paper_2510_26577_amd.device import to_device
    w = wl.random_workload(3, 2, 8, 2, 128, [700, 90], [9, 4])
    dw = to_device(w, "cuda:0")
    kw = dict(max_T=w.max_T, max_L=w.max_L, scale=w.scale, cu_L=dw.cu_L, parent=dw.parent)
    call = lambda **k: binding.tree_verify_attn(dw.q, dw.k_tree, dw.v_tree, dw.k_cache, dw.v_cache, None, dw.cu_T, dw.L, **{**kw, **k})
    o0, l0 = call()
    o, l = torch.empty_like(o0), torch.empty_like(l0)
    ws = torch.empty(1 << 20, dtype=torch.float32, device="cuda")
    o1, l1 = call(out=o, lse=l, workspace=ws, num_splits=3, L_host=list(map(int, w.L)), stream=torch.cuda.current_stream())
    assert o1 is o and l1 is l
    assert float((o1 - o0).abs().max()) < 2e-3 and float((l1 - l0).abs().max()) < 1e-4
    for bad, code in ((dict(scale=0.0), -1), (dict(max_T=200), -1), (dict(num_splits=-1), -1), (dict(cu_L=None), -1)):
        with pytest.raises(binding.TvaError) as e:
            call(**bad)
        assert e.value.code == code
    with pytest.raises(AssertionError):
        call(L_host=[1, 2, 3])
    with pytest.raises(TypeError):
        call(max_L=None)


def test_scratch_of_calls_on_another_stream_is_not_handed_out_while_they_wait():
    """Calls queued on a stream that is busy, from a program whose current stream is another: memory allocated and
    overwritten right behind them on the current stream must not be the scratch memory they are going to use."""
    import torch
    from oracle import verify_oracle as vo
    from paper_2510_26577_amd import binding, draft, verify, workloads as wl
    from paper_2510_26577_amd.device import to_device
    d = lambda x, t: torch.from_numpy(np.ascontiguousarray(x, dtype=t)).cuda()
    w = wl.random_workload(4, 1, 8, 2, 128, [3000], [9])
    dw = to_device(w, "cuda:0")
    rng = np.random.Generator(np.random.PCG64(31))
    cu_T, parent = np.array([0, 12], np.int32), wl.tree_expand_prune(rng, 12).astype(np.int32)
    p, q, tok, u, uf = wl.sampling_inputs(rng, parent, cu_T, 50000, drift=0.6)
    ref = vo.accept_sampling(parent, cu_T, tok, p, q, u, uf, max_path=8)
    scores = torch.rand((16, 145), device="cuda")
    cost = torch.cumsum(torch.full((72,), 0.03, dtype=torch.float64, device="cuda"), 0) + 4.0
    cu_N, score, logp = wl.expansion_inputs(rng, [5], 20000)
    sample = (d(parent, np.int32), d(cu_T, np.int32), d(tok, np.int32), d(p, np.float32), d(q, np.float32), d(u, np.float32), d(uf, np.float32), 8)
    grow = (d(cu_N, np.int32), d(score, np.float32), d(logp, np.float32), 8, 5)
    attn = dict(max_T=w.max_T, max_L=w.max_L, scale=w.scale, cu_L=dw.cu_L, parent=dw.parent, num_splits=8)
    calls = (lambda s: binding.tree_verify_attn(dw.q, dw.k_tree, dw.v_tree, dw.k_cache, dw.v_cache, None, dw.cu_T, dw.L, stream=s, **attn),
             lambda s: verify.accept_sampling(*sample, stream=s),
             lambda s: draft.rerank_count(scores, cost, 72, 1.0, stream=s), lambda s: draft.expand_layer(*grow, stream=s))
    want = [[t.clone() for t in c(None)] for c in calls]
    torch.cuda.synchronize()
    assert list(want[1][2].cpu().numpy()) == ref[1]
    side = torch.cuda.Stream()
    for c, expected in zip(calls, want):
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            torch.cuda._sleep(20_000_000)          # (some milliseconds)
        got = c(side)
        held = [torch.full((n,), float("nan"), device="cuda") for n in [64, 256, 1 << 10, 1 << 11, 1 << 12, 1 << 14, 1 << 16, 50000] for _ in range(8)]
        torch.cuda.synchronize()
        for g, e in zip(got, expected):
            assert torch.equal(g, e)
        del held

"""The library's helper streams with several threads: calls of one thread while
another captures a graph that uses a helper, and two threads at once.  Both fields
of a level on two streams are forced; results are those of one launch sequence."""
import sys
import threading

import numpy as np
import pytest

from sff_inputs import params_dict

pytestmark = pytest.mark.gpu

H, W, C = 53, 91, 3


def _calls(kind, seed):
    """A call of `kind` with its own tensors on a given stream, and a copy of its outputs."""
    import torch
    import paper_1710_10096_amd as sff
    rng = np.random.default_rng(seed)
    p = params_dict(H, W, C, levels=1, iters=3, fmax=16, dmax=12)
    dev = "cuda"
    imgs = torch.from_numpy(rng.integers(0, 256, (4, H, W, C), dtype=np.uint8)).to(dev)
    seeds = torch.tensor([seed], dtype=torch.int64, device=dev)
    hyp0 = torch.from_numpy(rng.integers(0, 13, (2, 1, H, W, 4)).astype(np.int16)).to(dev)
    if kind == "cost":
        feat = torch.from_numpy(rng.standard_normal((1, 4, H, W, 16)).astype(np.float32)).to(dev)
        w = torch.from_numpy(rng.random((1, H, W)).astype(np.float32)).to(dev)
        grad = torch.empty_like(feat)
        ws = torch.empty(sff.sff_cost_f32_bwd_workspace_bytes(1, H, W), dtype=torch.uint8, device=dev)
        outs = [grad]

        def run(stream):
            sff.sff_cost_f32_bwd(feat, hyp0[0], sff.DIR_FORWARD, w, grad_feat=grad, workspace=ws, stream=stream)
    else:
        bins = sff.sff_wht_features(p, imgs, 0, want_desc=False)
        desc = torch.from_numpy(rng.integers(-4000, 4001, (1, 4, H, W, 4, 16)).astype(np.int16)).to(dev)
        hyp = hyp0.clone()
        cost = torch.full((2, 1, H, W), -1, dtype=torch.int32, device=dev)
        outs = [hyp, cost]

        def run(stream):
            with torch.cuda.stream(stream):
                hyp.copy_(hyp0)
                cost.fill_(-1)
            if kind == "bins":
                sff.sff_match_level_bins(p, bins, sff.DIR_BOTH, 0, seeds, hyp, cost, stream=stream)
            else:
                sff.sff_match_level(p, desc, sff.DIR_BOTH, 0, seeds, hyp, cost, stream=stream)
    return run, lambda: [o.clone() for o in outs]


def _reference(kind, seed, monkeypatch):
    import torch
    run, out = _calls(kind, seed)
    with monkeypatch.context() as m:
        m.setenv("SFF_MATCH_SPLIT", "0")
        m.setenv("SFF_COST_F32_SPLIT", "0")
        run(torch.cuda.current_stream())
    torch.cuda.synchronize()
    return out()


def _same(a, b):
    import torch
    return all(torch.equal(x, y) for x, y in zip(a, b))


KINDS = ["bins", "records", "cost"]


@pytest.mark.parametrize("other", KINDS)
@pytest.mark.parametrize("captured", KINDS)
def test_calls_beside_a_capture(captured, other, monkeypatch):
    import torch
    print("[case] helper streams, capture of", captured, "beside", other, file=sys.stderr, flush=True)
    want_a, want_b = _reference(captured, 1, monkeypatch), _reference(other, 2, monkeypatch)
    monkeypatch.setenv("SFF_MATCH_SPLIT", "1")
    run_a, out_a = _calls(captured, 1)
    run_b, out_b = _calls(other, 2)
    s, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    run_a(s)
    torch.cuda.synchronize()
    failed = []

    def beside():
        try:
            run_b(s2)
        except Exception as e:  # noqa: BLE001 -- reported by the test's thread
            failed.append(e)

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s, capture_error_mode="thread_local"):
        run_a(s)
        t = threading.Thread(target=beside)
        t.start()
        t.join()
        run_a(s)
    torch.cuda.synchronize()
    assert not failed, failed
    assert _same(out_b(), want_b)
    for _ in range(3):
        g.replay()
        run_b(s2)
        torch.cuda.synchronize()
        assert _same(out_a(), want_a) and _same(out_b(), want_b)


def test_two_threads_at_once(monkeypatch):
    import torch
    print("[case] helper streams, two threads", file=sys.stderr, flush=True)
    want = {k: _reference(k, 3 + i, monkeypatch) for i, k in enumerate(KINDS)}
    monkeypatch.setenv("SFF_MATCH_SPLIT", "1")
    bad = []

    def work(kinds):
        try:
            s = torch.cuda.Stream()
            calls = {k: _calls(k, 3 + KINDS.index(k)) for k in kinds}
            torch.cuda.synchronize()
            for _ in range(20):
                for run, _o in calls.values():
                    run(s)
            s.synchronize()
            bad.extend(k for k in kinds if not _same(calls[k][1](), want[k]))
        except Exception as e:  # noqa: BLE001
            bad.append(e)

    ts = [threading.Thread(target=work, args=(KINDS[i:] + KINDS[:i],)) for i in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad

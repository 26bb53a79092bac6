"""One-shot calls in flight on several streams and threads at once: their
tables come from a bounded pool of slots that is handed round many times, and
every call's result equals the plan's, bit for bit."""
import threading

import pytest
import torch

from paper_2607_02945_amd import binding as B
from paper_2607_02945_amd import synth
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def _group(seed, G, M):
    g = synth.rng(seed)
    mk = lambda *s: synth.to_storage(g.standard_normal(s), "bf16").to("cuda")
    Ks, Ns = g.integers(8, 200, G).tolist(), g.integers(8, 200, G).tolist()
    return [mk(M, k) for k in Ks], [mk(n, k) for n, k in zip(Ns, Ks)], [mk(n) for n in Ns]


@pytest.mark.parametrize("threads,M", [(1, 64), (4, 64), (3, 3000)])  # 3000 rows: tables past a slot's size
def test_many_calls_in_flight(threads, M):
    say(f"[one-shot] threads={threads} M={M}")
    errors = []

    def work(i):
        try:
            stream = torch.cuda.Stream()
            groups = [_group(100 * i + j, 5 + 11 * j, M) for j in range(3)]
            refs, outs = [], []
            for xs, ws, bs in groups:
                y = [torch.empty(M, w.shape[0], dtype=x.dtype, device="cuda") for x, w in zip(xs, ws)]
                t = [torch.empty_like(v) for v in y]
                B.optimus_plan_linear(xs, ws, bs, y, "relu").execute()
                B.optimus_plan_pointwise(y, t, "tanh").execute()
                refs.append((y, t))
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                for rep in range(60):
                    xs, ws, bs = groups[rep % 3]
                    y = [torch.full_like(v, float("nan")) for v in refs[rep % 3][0]]
                    t = [torch.full_like(v, float("nan")) for v in y]
                    B.optimus_grouped_linear(xs, ws, bs, y, "relu")
                    B.optimus_grouped_pointwise(y, t, "tanh")
                    outs.append((rep % 3, y, t))
                stream.synchronize()
            for k, y, t in outs:
                for a, b in zip(y + t, refs[k][0] + refs[k][1]):
                    assert torch.equal(a, b), f"thread {i} group {k}"
        except Exception as e:  # reported by the main thread
            errors.append(e)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors[0]

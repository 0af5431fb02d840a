"""A step on a given x that nobody waits for: the call enqueues the logits alone, spread over several compute units, and every
workgroup of the expert launch routes for itself.  Bit for bit against the step that is waited for, where one kernel does both."""
import pytest
import torch

from synth import workloads
from synth.workloads import CONFIGS

from _gpu_common import DEV, build

pytestmark = pytest.mark.gpu

C2 = CONFIGS["c2_qwen_bf16"]


def config(fmt, hidden, n_experts):
    return C2.with_(n_layers=2, hidden=hidden, inter=128, shared_inter=0, n_experts=n_experts, capacity=max(3, n_experts // 2),
                    top_k=3, weight_fmt=fmt, act_fmt="fp32" if fmt == "fp32" else "bf16", seed=9100 + hidden + n_experts)


SHAPES = [("fp32", 256, 5), ("fp32", 1024, 64), ("bf16", 512, 4), ("bf16", 1024, 7), ("int8", 2048, 61), ("int8", 4096, 9),
          ("fp32", 2048, 6)]


def record(dec, layer, k, n_experts):
    r = dec.last_route(layer)
    return [list(r.sel_expert)[:k], list(r.sel_weight)[:k], list(r.sel_slot)[:k], list(r.logits)[:n_experts]]


@pytest.mark.parametrize("fmt,hidden,n_experts", SHAPES)
def test_step_on_a_given_x(fmt, hidden, n_experts, monkeypatch):
    monkeypatch.setenv("MOE_ROUTE_EVERYWHERE", "1")
    cfg = config(fmt, hidden, n_experts)
    print(f"case step on a given x {fmt} hidden={hidden} experts={n_experts}", flush=True)
    a = workloads.ar1_stream(cfg, 5).to(cfg.act_dtype).to(DEV)
    got = []
    for wait in (True, False):
        _, dec = build(cfg, lam=0.3)
        y = torch.zeros((5, 2, hidden), dtype=cfg.act_dtype, device=DEV)
        recs = []
        torch.cuda.synchronize()
        for t in range(5):
            for l in range(2):
                dec.route_step(l, x=a[t, l], wait=wait)
                dec.expert_forward(l, a[t, l], y[t, l])
                recs.append(record(dec, l, cfg.top_k, n_experts))
        torch.cuda.synchronize()
        got.append((y.cpu(), recs))
    assert got[0][1] == got[1][1]
    assert torch.equal(got[0][0], got[1][0])

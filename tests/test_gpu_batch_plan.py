"""Batches routed from x have their expert kernels enqueued behind the routing, with a list of experts made on the device;
batches routed from logits (and those in which something misses, or whose list is too long) get it from the host.  The same
tokens both ways, at the sizes where the list changes: one token, several groups of 64 tokens per expert, all slots in use,
with and without a shared expert, units of one and of several rounds.  The lists are equal, so the outputs are bit for bit."""
import pytest
import torch

from synth import workloads
from synth.workloads import CONFIGS

from _gpu_common import DEV, build

pytestmark = pytest.mark.gpu

C2 = CONFIGS["c2_qwen_bf16"]


@pytest.mark.parametrize("hidden,inter,shared,N,K,C,tokens", [
    (1024, 16, 0, 4, 1, 4, 1), (1024, 48, 32, 4, 2, 4, 128), (2048, 160, 208, 64, 8, 64, 128), (1024, 96, 0, 64, 8, 64, 65),
    (2048, 1056, 16, 3, 2, 3, 100), (1024, 4096, 2048, 6, 4, 6, 33), (1024, 208, 6000, 16, 3, 16, 16), (2048, 512, 0, 40, 8, 40, 64)])
def test_lists_of_device_and_host_are_the_same(hidden, inter, shared, N, K, C, tokens):
    cfg = C2.with_(n_layers=1, hidden=hidden, inter=inter, shared_inter=shared, n_experts=N, capacity=C, top_k=K, seed=9100 + inter)
    print(f"case batch plan d={hidden} I={inter} shared={shared} N={N} K={K} C={C} tokens={tokens}", flush=True)
    ids = [list(range(C))]
    store, a = build(cfg, lam=0.5, initial=ids)
    import paper_2412_00099_amd as pkg

    b = pkg.MoEDecoder(store, top_k=K, lam=0.5, initial=ids)
    xs = workloads.ar1_stream(cfg, 2 * tokens)[:, 0].to(cfg.act_dtype).to(DEV)
    out = torch.zeros(4, tokens, hidden, dtype=cfg.act_dtype, device=DEV)
    torch.cuda.synchronize()
    for i in range(2):  # (other tokens behind the first: the list is made anew)
        x = xs[i * tokens:(i + 1) * tokens]
        recs = a.route_batch(0, x=x)
        a.expert_forward_batch(0, x, out[2 * i])
        assert all(r.n_miss == 0 for r in recs)
        logits = torch.tensor([[r.logits[e] for e in range(N)] for r in recs], dtype=torch.float32).to(DEV)
        torch.cuda.synchronize()
        b.route_batch(0, logits=logits)
        b.expert_forward_batch(0, x, out[2 * i + 1])
    assert torch.equal(out[0], out[1]) and torch.equal(out[2], out[3])
    assert float(out.float().abs().max()) > 0
    # another x than the one that was routed: computed with what is given
    a.route_batch(0, x=xs[:tokens])
    other = xs[tokens:].clone()
    a.expert_forward_batch(0, other, out[0])
    b.route_batch(0, x=xs[:tokens])
    b.expert_forward_batch(0, other, out[1])
    y = torch.zeros_like(out[2])
    b.route_batch(0, x=xs[:tokens])
    b.expert_forward_batch(0, xs[:tokens], y)
    assert torch.equal(out[0], out[1]) and not torch.equal(out[0], y)
    a.close()
    b.close()

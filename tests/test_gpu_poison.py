"""Use-before-fill guard.  Fills by the host: with MOE_POISON_FILLS=1 the library overwrites a slot with NaN patterns right
before the copy that fills it.  Fills by the expert launch (which that switch turns off): the slots hold NaN patterns when the
decoder is made.  A kernel that computed from a slot before its fill had landed would put NaNs into y, which the output
comparisons of these runs (misses on most tokens: small caches) cannot pass."""
import pytest
import torch

import paper_2412_00099_amd as pkg
import test_gpu_route
import test_gpu_stack
from synth.workloads import CONFIGS

from test_gpu_prompt import run_prompt_outputs
from test_gpu_stack import run_in_launch_boundary

pytestmark = pytest.mark.gpu


def poisoned_slots(monkeypatch, module, form=pkg.MOE_FILLS_IN_EXPERT_LAUNCH):
    """Decoders that `module` makes from here on start from slots full of NaN patterns and fill them as `form` says."""
    plain = module.build

    def build(cfg, **kw):
        store, dec = plain(cfg, **kw)
        assert dec.fill_form() == form
        store.pools.fill_(0xff)
        torch.cuda.synchronize()
        return store, dec

    monkeypatch.setattr(module, "build", build)


@pytest.mark.parametrize("name,hidden,inter", [("c2_qwen_bf16", 2048, 96), ("c4_dsv2lite_int4", 2048, 128),
                                               ("c5_mixtral_int8", 1024, 64)])
def test_decode_with_poisoned_fills(name, hidden, inter, monkeypatch):
    monkeypatch.setenv("MOE_POISON_FILLS", "1")
    poisoned_slots(monkeypatch, test_gpu_stack, form=pkg.MOE_FILLS_BY_HOST)
    base = CONFIGS[name]
    cfg = base.with_(n_layers=2, hidden=hidden, n_experts=12, inter=inter,
                     shared_inter=2 * inter if base.shared_inter else 0, capacity=5, top_k=min(base.top_k, 4),
                     seed=7700 + hidden + inter)
    ties, misses = run_in_launch_boundary(cfg, 12, 0.0, monkeypatch=monkeypatch)
    assert misses > cfg.top_k * cfg.n_layers  # LRU routing on a cache of five: refills well beyond the cold ones


@pytest.mark.parametrize("boundary", ["first workgroup", "every workgroup", "own launch"])
@pytest.mark.parametrize("name,hidden,inter", [("c2_qwen_bf16", 2048, 96), ("c4_dsv2lite_int4", 2048, 128),
                                               ("c5_mixtral_int8", 1024, 64)])
def test_decode_into_poisoned_slots(name, hidden, inter, boundary, monkeypatch):
    """The launch that fills slots, in every form of the boundary."""
    base = CONFIGS[name]
    cfg = base.with_(n_layers=2, hidden=hidden, n_experts=12, inter=inter,
                     shared_inter=2 * inter if base.shared_inter else 0, capacity=5, top_k=min(base.top_k, 4),
                     seed=7900 + hidden + inter)
    if boundary == "first workgroup":
        poisoned_slots(monkeypatch, test_gpu_stack)
        ties, misses = run_in_launch_boundary(cfg, 12, 0.0, monkeypatch=monkeypatch)
        assert misses > cfg.top_k * cfg.n_layers
    else:
        monkeypatch.setenv("MOE_FUSE_BOUNDARY", "0")
        monkeypatch.setenv("MOE_ROUTE_EVERYWHERE", "1" if boundary == "every workgroup" else "0")
        poisoned_slots(monkeypatch, test_gpu_route)
        test_gpu_route.free_run(cfg, 0.0, 12, deferred=True)


def test_prompt_phase_with_poisoned_fills(monkeypatch):
    monkeypatch.setenv("MOE_POISON_FILLS", "1")
    cfg = CONFIGS["c2_qwen_bf16"].with_(n_layers=1, hidden=1024, n_experts=10, inter=48, shared_inter=96, top_k=2,
                                        capacity=3, seed=7801)
    run_prompt_outputs(cfg, 0.0, [8, 37, 128, 16])

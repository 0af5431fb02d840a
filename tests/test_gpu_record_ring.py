"""The record ring of the expert kernels at the sizes where its places and blocks change: one record per wavefront, one
more and one less, places that stay empty, lists of shared records only in some workgroups, d = 4096 with one record in
flight, and every combination with experts that are filled for the token (second launch).  Against the oracle, with its
output tolerances (1e-5 fp32, 1e-2 bf16: the rounding of y is 2^-8 at most)."""
import pytest

from synth.workloads import CONFIGS

from test_gpu_route import free_run

C1 = CONFIGS["c1_single_fp32"]
C2 = CONFIGS["c2_qwen_bf16"]


def test_record_split_by_multiplication():
    # kernels split n = q G + r records over G <= 1024 workgroups with (b r * ceil(2^32 / G)) >> 32 for floor(b r / G)
    for G in range(1, 1025):
        inv = (((1 << 32) + G - 1) // G) & 0xFFFFFFFF
        for r in {0, 1, G // 2, G - 1} - {G}:
            for b in {0, 1, G // 3, G - 1, G}:
                assert (b * r * inv) >> 32 == b * r // G, (G, r, b)


# 256 workgroups x 8 wavefronts = 2048 places of one record
@pytest.mark.gpu
@pytest.mark.parametrize("inter,shared", [(1024, 0), (1023, 1), (1025, 0), (2048, 3), (128, 1793)])
def test_blocks_of_two_records(inter, shared):
    cfg = C1.with_(inter=inter, shared_inter=shared, n_experts=5, capacity=3, seed=700 + inter)
    print(f"case ring fp32 inter={inter} shared={shared}", flush=True)
    free_run(cfg, 0.0, 10)
    free_run(cfg, 0.0, 6, deferred=True)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,hidden,inter,shared", [
    ("bf16", 4096, 130, 33), ("bf16", 1024, 1025, 0), ("fp32", 2048, 300, 77), ("int8", 1024, 1032, 8),
    ("int8", 2048, 1016, 520), ("int8", 4096, 264, 0), ("int4", 2048, 128, 0), ("int4", 2048, 1152, 128),
    ("int4", 4096, 384, 256)])
def test_every_format(fmt, hidden, inter, shared):
    act = "fp32" if fmt == "fp32" else "bf16"
    cfg = C2.with_(n_layers=1, hidden=hidden, inter=inter, shared_inter=shared, n_experts=4, capacity=3, top_k=2,
                   weight_fmt=fmt, act_fmt=act, seed=800 + hidden + inter)
    print(f"case ring {fmt} hidden={hidden} inter={inter} shared={shared}", flush=True)
    free_run(cfg, 0.0, 6)
    free_run(cfg, 0.0, 4, deferred=True)

"""Experts that miss in a step nobody waits for are brought in by the expert launch itself: they are computed while they are
streamed from the host tier and put into their slots on the way.  Against the oracle in every form of the boundary, with
frequent misses and a cache of few slots, so that what was put into a slot (records, row scales, down scales) is computed
with afterwards; and slot by slot against the host tier, byte for byte."""
import numpy as np
import pytest
import torch

import paper_2412_00099_amd as pkg
from synth import workloads
from synth.workloads import CONFIGS

import test_gpu_route
from _gpu_common import DEV, build
from test_gpu_poison import poisoned_slots
from test_gpu_route import free_run

pytestmark = pytest.mark.gpu

C2 = CONFIGS["c2_qwen_bf16"]
C4 = CONFIGS["c4_dsv2lite_int4"]
SHAPES = [("fp32", 256, 96, 0), ("fp32", 2048, 40, 24), ("bf16", 512, 300, 0), ("bf16", 2048, 264, 88), ("bf16", 4096, 72, 0),
          ("int8", 1024, 520, 0), ("int8", 2048, 264, 40), ("int8", 4096, 8, 0), ("int4", 2048, 384, 128), ("int4", 4096, 256, 0)]


def config(fmt, hidden, inter, shared):
    return C2.with_(n_layers=2, hidden=hidden, inter=inter, shared_inter=shared, n_experts=9, capacity=4, top_k=3,
                    weight_fmt=fmt, act_fmt="fp32" if fmt == "fp32" else "bf16", seed=8100 + hidden + inter)


def used_bytes(cfg, store):
    """Blob bytes that mean something: int4 records and blobs end in padding."""
    d, I = cfg.hidden, cfg.inter
    mask = np.ones(store.blob_bytes, bool)
    if cfg.weight_fmt == "int4":
        rec = 3 * (d // 2) + ((d // 128) * 4 + 127) // 128 * 128
        for i in range(I):
            mask[i * rec + 3 * (d // 2) + (d // 128) * 4:(i + 1) * rec] = False
        mask[I * rec + I // 128 * d * 2:] = False
    else:
        rec = 3 * d * {"fp32": 4, "bf16": 2, "int8": 1}[cfg.weight_fmt]
        mask[I * rec + (4 * I + 2 * d if cfg.weight_fmt == "int8" else 0):] = False
    return mask


@pytest.mark.parametrize("everywhere", ["0", "1"])
@pytest.mark.parametrize("fmt,hidden,inter,shared", SHAPES)
def test_slots_hold_the_host_tiers_bytes(fmt, hidden, inter, shared, everywhere, monkeypatch):
    monkeypatch.setenv("MOE_ROUTE_EVERYWHERE", everywhere)
    monkeypatch.setenv("MOE_FUSE_BOUNDARY", "0")
    cfg = config(fmt, hidden, inter, shared)
    print(f"case device fills {fmt} hidden={hidden} inter={inter} everywhere={everywhere}", flush=True)
    store, dec = build(cfg, lam=0.0)
    assert dec.fill_form() == pkg.MOE_FILLS_IN_EXPERT_LAUNCH
    h = torch.zeros(hidden, device=DEV)
    x = torch.zeros(hidden, dtype=cfg.act_dtype, device=DEV)
    y = torch.zeros_like(x)
    a = workloads.ar1_stream(cfg, 6).to(DEV)
    torch.cuda.synchronize()
    for t in range(6):
        for l in range(cfg.n_layers):
            dec.stack_route_step(l, h, a[t, l], 1.0 if l == 0 else 0.5, x, carry=l > 0, wait=False)
            dec.expert_forward(l, x, y if l == cfg.n_layers - 1 else None)
    st = dec.stats()
    assert st.misses > cfg.top_k * cfg.n_layers and st.bytes_filled == st.misses * store.blob_bytes
    mask = used_bytes(cfg, store)
    for l in range(cfg.n_layers):
        tables = dec.tables(l)
        pool = store.pools[l].cpu().numpy().reshape(cfg.capacity, store.blob_bytes)
        for s in range(cfg.capacity):
            e = tables.slot_expert[s]
            if e >= 0:
                assert np.array_equal(pool[s][mask], store.host[l, e].numpy()[mask]), (l, s, e)
    dec.close()


@pytest.mark.parametrize("N,K,C,n_initial,mode,top_j", [(64, 8, 8, 0, 0, 0), (64, 8, 13, 5, 0, 2), (61, 7, 9, 9, 1, 1),
                                                      (60, 8, 11, 4, 2, 0), (8, 1, 1, 0, 0, 0), (64, 5, 64, 20, 0, 0)])
def test_every_workgroup_finds_the_slots_by_itself(N, K, C, n_initial, mode, top_j, monkeypatch):
    """Where the routing is left to every workgroup, each works out into which slots the missing experts go; it does not wait
    for the first one to say so (a limit of one poll changes nothing).  Empty slots, evictions and both at once, in every
    routing mode: pools as the first workgroup's tables say, outputs and counters as with fills by the host."""
    cfg = C2.with_(n_layers=1, hidden=512, inter=24, shared_inter=0, n_experts=N, capacity=C, top_k=K, seed=8500 + N + C)
    print(f"case slots found in every workgroup N={N} K={K} C={C} initial={n_initial} mode={mode}", flush=True)
    monkeypatch.setenv("MOE_FUSE_BOUNDARY", "0")
    monkeypatch.setenv("MOE_ROUTE_EVERYWHERE", "1")
    monkeypatch.setenv("MOE_TAG_SPINS", "1")
    out = []
    for on in ("1", "0"):
        monkeypatch.setenv("MOE_DEVICE_FILLS", on)
        store, dec = build(cfg, lam=0.1, top_j=top_j, initial=[list(range(N))[N - n_initial:]] if n_initial else None,
                           route_mode=mode, max_rank=min(2 * K, N), cumsum_p=0.5)
        assert dec.fill_form() == int(on)
        xs = workloads.ar1_stream(cfg, 24)[:, 0].to(cfg.act_dtype).to(DEV)
        ys = torch.zeros_like(xs)
        torch.cuda.synchronize()
        for t in range(24):
            dec.route_step(0, x=xs[t], wait=False)
            dec.expert_forward(0, xs[t], ys[t])
        tables, st = dec.tables(0), dec.stats(0)
        assert st.misses >= 5
        pool = store.pools[0].cpu().numpy().reshape(C, store.blob_bytes)
        for s in range(C):
            e = tables.slot_expert[s]
            assert e < 0 or np.array_equal(pool[s], store.host[0, e].numpy()), (s, e)
        out.append((ys.cpu(), bytes(tables), bytes(st)))
        dec.close()
    assert torch.equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]


@pytest.mark.parametrize("fmt,hidden,inter,shared", SHAPES)
def test_outputs(fmt, hidden, inter, shared, monkeypatch):
    """(What the slots hold at first would make y NaN: an expert's record is used before it is in its slot by nobody.)"""
    cfg = config(fmt, hidden, inter, shared)
    print(f"case device fills outputs {fmt} hidden={hidden} inter={inter}", flush=True)
    poisoned_slots(monkeypatch, test_gpu_route)
    free_run(cfg, 0.0, 10, deferred=True)


@pytest.mark.parametrize("env", [dict(MOE_FUSE_BOUNDARY="1"), dict(MOE_FUSE_BOUNDARY="0", MOE_ROUTE_EVERYWHERE="1"),
                                 dict(MOE_FUSE_BOUNDARY="0", MOE_ROUTE_EVERYWHERE="0")])
@pytest.mark.parametrize("fmt", ["bf16", "int8", "int4"])
def test_same_outputs_as_with_fills_by_the_host(fmt, env, monkeypatch):
    """In every form of the boundary: outputs to bf16 rounding (with the boundary in the first workgroup the two ways split the
    records that missed over 255 and over 256 workgroups; the other two forms are bit for bit, see below), decisions the same."""
    cfg = (C4 if fmt == "int4" else C2).with_(n_layers=2, hidden=2048, inter=384, shared_inter=512, n_experts=12, capacity=5,
                                              top_k=4, weight_fmt=fmt, seed=8200)
    print(f"case device fills against host fills {fmt} {env}", flush=True)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    out = []
    for on in ("1", "0"):
        monkeypatch.setenv("MOE_DEVICE_FILLS", on)
        store, dec = build(cfg, lam=0.0)
        assert dec.fill_form() == int(on)
        h = torch.zeros(cfg.hidden, device=DEV)
        x = torch.zeros(cfg.hidden, dtype=cfg.act_dtype, device=DEV)
        a = workloads.ar1_stream(cfg, 8).to(DEV)
        ys = torch.zeros(8, 2, cfg.hidden, dtype=cfg.act_dtype, device=DEV)
        torch.cuda.synchronize()
        for t in range(8):
            for l in range(2):  # (a new residual stream in every layer: a rounding does not travel)
                dec.stack_route_step(l, h, a[t, l], 1.0, x, carry=False, wait=False)
                dec.expert_forward(l, x, ys[t, l])
        st = dec.stats()
        out.append((ys.float().cpu(), bytes(dec.tables(0)), bytes(dec.tables(1)), bytes(st)))
        dec.close()
    assert out[0][1:] == out[1][1:]
    scale = out[1][0].abs().amax(dim=2, keepdim=True)
    assert float(((out[0][0] - out[1][0]).abs() / scale).max()) <= 2.0 ** -7  # two roundings to bf16


@pytest.mark.parametrize("everywhere", ["0", "1"])
@pytest.mark.parametrize("fmt,shared,inter", [("fp32", 200, 300), ("bf16", 520, 384), ("int8", 264, 1016), ("int4", 640, 1152)])
def test_bit_for_bit_as_with_fills_by_the_host(fmt, shared, inter, everywhere, monkeypatch):
    """With the boundary ahead of the expert launch the launch's second walk adds the same products in the same order as the
    second launch behind fills by the host, beside a shared expert too."""
    cfg = C2.with_(n_layers=2, hidden=2048, inter=inter, shared_inter=shared, n_experts=12, capacity=5, top_k=4, weight_fmt=fmt,
                   act_fmt="fp32", seed=8300 + inter)
    print(f"case device fills bit for bit {fmt} everywhere={everywhere}", flush=True)
    monkeypatch.setenv("MOE_FUSE_BOUNDARY", "0")
    monkeypatch.setenv("MOE_ROUTE_EVERYWHERE", everywhere)
    out = []
    for on in ("1", "0"):
        monkeypatch.setenv("MOE_DEVICE_FILLS", on)
        store, dec = build(cfg, lam=0.0)
        assert dec.fill_form() == int(on)
        h = torch.zeros(cfg.hidden, device=DEV)
        x = torch.zeros(cfg.hidden, dtype=cfg.act_dtype, device=DEV)
        a = workloads.ar1_stream(cfg, 8).to(DEV)
        ys = torch.zeros(8, 2, cfg.hidden, dtype=cfg.act_dtype, device=DEV)
        torch.cuda.synchronize()
        for t in range(8):
            for l in range(2):
                dec.stack_route_step(l, h, a[t, l], 1.0 if l == 0 else 0.5, x, carry=l > 0, wait=False)
                dec.expert_forward(l, x, ys[t, l])
        st = dec.stats()
        assert st.misses > 3 * cfg.top_k
        out.append((ys.cpu(), bytes(st)))
        dec.close()
    assert torch.equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]


def test_host_tier_that_is_not_pinned(monkeypatch):
    """The launch cannot read such memory: the host enqueues the fills, as it does where it waits for the decision."""
    cfg = config("bf16", 1024, 96, 32)
    print("case host tier not pinned", flush=True)
    out = []
    for pinned in (True, False):
        store, dec = build(cfg, lam=0.0)
        if not pinned:
            dec.close()
            store.host = store.host.clone()
            assert not store.host.is_pinned()
            dec = pkg.MoEDecoder(store, top_k=cfg.top_k)
        assert dec.fill_form() == (pkg.MOE_FILLS_IN_EXPERT_LAUNCH if pinned else pkg.MOE_FILLS_BY_HOST)
        xs = workloads.ar1_stream(cfg, 8)[:, 0].to(cfg.act_dtype).to(DEV)
        ys = torch.zeros_like(xs)
        torch.cuda.synchronize()
        for t in range(8):
            dec.route_step(0, x=xs[t], wait=False)
            dec.expert_forward(0, xs[t], ys[t])
        dec.compute_stream.synchronize()
        out.append((ys.cpu(), bytes(dec.tables(0)), bytes(dec.stats(0))))
        dec.close()
    assert torch.equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]


def test_a_step_is_not_captured():
    cfg = config("bf16", 1024, 96, 32)
    print("case capture refused", flush=True)
    store, dec = build(cfg, lam=0.0)
    assert dec.fill_form() == pkg.MOE_FILLS_IN_EXPERT_LAUNCH
    x = torch.randn(1024, device=DEV).to(torch.bfloat16)
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(dec.compute_stream):
        graph.capture_begin(capture_error_mode="relaxed")
        dec.route_step(0, x=x, wait=False)
        with pytest.raises(pkg.MoEError):
            dec.expert_forward(0, x, y)
        graph.capture_end()
    dec.reset()
    dec.route_step(0, x=x, wait=False)
    dec.expert_forward(0, x, y)
    dec.compute_stream.synchronize()
    assert float(y.float().abs().max()) > 0
    dec.close()


def test_the_callers_logits_are_the_callers_again():
    """A step on given logits that nobody waits for: moe_expert_forward returns once they have been read, so a caller may
    put the next token's into the same buffer, from any stream.  (The stream is held by a kernel of a fixed length.)"""
    cfg = config("bf16", 1024, 96, 32)
    print("case logits refilled behind moe_expert_forward", flush=True)
    store, dec = build(cfg, lam=0.0)
    zs = workloads.logits_stream(cfg, 5, layer=0, scale=2.0).to(DEV)
    z = torch.zeros_like(zs[0])
    x = torch.randn(1024, device=DEV).to(torch.bfloat16)
    y = torch.zeros_like(x)
    for t in range(5):
        z.copy_(zs[t])
        torch.cuda.synchronize()
        with torch.cuda.stream(dec.compute_stream):
            torch.cuda._sleep(20_000_000)
        dec.route_step(0, logits=z, wait=False)
        dec.expert_forward(0, x, y)
        z.fill_(-1.0)
        torch.cuda.current_stream().synchronize()
        want = torch.sort(zs[t], descending=True).indices[:cfg.top_k].tolist()
        assert list(dec.last_route(0).sel_expert[:cfg.top_k]) == want
    dec.close()


def test_a_temporary_a_is_not_given_out_again():
    """The residual input of a boundary that nobody waits for is a temporary of the caller's: its memory stays its own until
    the kernel that reads it has run."""
    cfg = config("bf16", 1024, 96, 32)
    print("case temporary a", flush=True)
    a = workloads.ar1_stream(cfg, 1).to(DEV)[0, 0]
    out = []
    for hold in (False, True):
        store, dec = build(cfg, lam=0.0)
        h = torch.zeros(1024, device=DEV)
        x = torch.zeros(1024, dtype=torch.bfloat16, device=DEV)
        y = torch.zeros_like(x)
        torch.cuda.synchronize()
        temporary = a * 2.0
        torch.cuda.synchronize()
        if hold:
            with torch.cuda.stream(dec.compute_stream):
                torch.cuda._sleep(20_000_000)
        dec.stack_route_step(0, h, temporary, 1.0, x, carry=False, wait=False)
        dec.expert_forward(0, x, y)
        del temporary
        others = [torch.full((1024,), 7.0, device=DEV) for _ in range(64)]
        torch.cuda.synchronize()
        out.append((h.cpu(), y.cpu()))
        del others
        dec.close()
    assert torch.equal(out[0][0], (a * 2.0).cpu()) and torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])

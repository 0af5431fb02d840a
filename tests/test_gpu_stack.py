"""The fused layer boundary (pending expert output + residual/normalisation glue + routing in one launch)
against the oracle, through the C ABI."""
import numpy as np
import pytest
import torch

from oracle import experts as oexp
from oracle import routing, stack
from synth import workloads
from synth.workloads import CONFIGS

from _gpu_common import DEV, OracleWeights, build, route_fields

pytestmark = pytest.mark.gpu


def test_coupled_fp32_stack_fused_boundary():
    """Three coupled fp32 layers, 24 tokens: x of every layer, every routing decision and the final hidden state."""
    cfg = CONFIGS["c1_single_fp32"].with_(n_layers=3, inter=96, shared_inter=64, seed=707)
    L, K, N, d, T, lam = cfg.n_layers, cfg.top_k, cfg.n_experts, cfg.hidden, 24, 0.5
    store, dec = build(cfg, lam=lam)
    ow = OracleWeights(cfg)
    routers = [routing.CachePriorRouter(N, K, cfg.capacity, lam) for _ in range(L)]
    a = workloads.ar1_stream(cfg, T)
    a_dev = a.to(DEV)
    h = torch.zeros(d, device=DEV)
    xs = torch.zeros(L, d, device=DEV)
    y_last = torch.zeros(d, device=DEV)
    torch.cuda.synchronize()
    ties = 0
    for t in range(T):
        h_ref = a[t, 0].double().numpy()
        for l in range(L):
            raw = dec.stack_route_step(l, h, a_dev[t, l], 1.0 if l == 0 else stack.PERTURB, xs[l], carry=l > 0,
                                       y=y_last if l == 0 else None)
            dec.expert_forward(l, xs[l], None)  # output stays pending as partial rows
            dec.compute_stream.synchronize()
            out = route_fields(raw, K)
            x_ref = stack.rmsnorm(h_ref).astype(np.float32)
            assert oexp.rel_err(xs[l].cpu().numpy(), x_ref) <= 2e-6, (t, l)
            z = routing.router_logits(ow.gate(l), x_ref)
            sel, zp, delta = routers[l].select(z)
            if out["sel"] != sel.tolist():
                kth = np.sort(zp)[::-1][K - 1]
                assert np.all(zp[out["sel"]] >= kth - 1e-5), (t, l, out["sel"], sel.tolist())
                ties += 1
                sel = np.array(out["sel"])
            ref = routers[l].commit(z, sel, zp, delta)
            assert out["slot"] == ref.slot and out["miss"] == ref.miss, (t, l)
            y_ref = oexp.moe_output(x_ref, [ow.expert(l, int(e)) for e in ref.sel], ref.weight, ow.shared(l))
            if l + 1 < L:
                h_ref = stack.next_hidden(h_ref, y_ref, a[t, l + 1].numpy())
        y_prev_ref = y_ref  # the last layer's output stays pending until the next boundary call
    # flush: one more boundary call hands out the pending output of the very last layer
    dec.stack_route_step(0, h, a_dev[0, 0], 1.0, xs[0], carry=False, y=y_last)
    dec.expert_forward(0, xs[0], None)
    dec.compute_stream.synchronize()
    assert oexp.rel_err(y_last.cpu().numpy(), y_prev_ref) <= 1e-5
    for l in range(L):
        s, o = dec.stats(l), routers[l].stats
        if l > 0:
            assert (s.tokens, s.hits, s.misses) == (o.tokens, o.hits, o.misses)
    print(f"coupled fp32 stack: ties={ties}", flush=True)
    dec.close()


@pytest.mark.parametrize("name,hidden", [("c2_qwen_bf16", 2048), ("c2_qwen_bf16", 4096), ("c1_single_fp32", 256)])
def test_fused_boundary_single_step(name, hidden):
    """route + experts of layer 0 on a seeded x0, then the fused boundary of layer 1 on seeded h, a."""
    base = CONFIGS[name]
    cfg = base.with_(n_layers=2, hidden=hidden, n_experts=12, inter=128, shared_inter=128 if base.shared_inter else 0,
                     capacity=6, top_k=min(base.top_k, 4), seed=900 + hidden)
    K, N, d = cfg.top_k, cfg.n_experts, cfg.hidden
    store, dec = build(cfg, lam=0.5)
    ow = OracleWeights(cfg)
    a = workloads.ar1_stream(cfg, 3)
    x0 = a[0, 0].to(cfg.act_dtype)
    h0, a1 = a[1, 0].clone(), a[2, 1].clone()
    x0d, hd, ad = x0.to(DEV), h0.to(DEV), a1.to(DEV)
    x1d = torch.zeros(d, dtype=cfg.act_dtype, device=DEV)
    yd = torch.zeros(d, dtype=cfg.act_dtype, device=DEV)
    torch.cuda.synchronize()
    r0 = route_fields(dec.route_step(0, x=x0d), K)
    dec.expert_forward(0, x0d, None)
    r1 = dec.stack_route_step(1, hd, ad, stack.PERTURB, x1d, carry=True, y=yd)
    dec.expert_forward(1, x1d, None)
    dec.compute_stream.synchronize()
    x0n = x0.float().numpy()
    router0 = routing.CachePriorRouter(N, K, cfg.capacity, 0.5)
    ref0 = router0.step(routing.router_logits(ow.gate(0), x0n))
    assert r0["sel"] == ref0.sel.tolist()
    y_ref = oexp.moe_output(x0n, [ow.expert(0, int(e)) for e in ref0.sel], ref0.weight, ow.shared(0))
    tol = 1e-5 if cfg.act_fmt == "fp32" else 1e-2
    assert oexp.rel_err(yd.float().cpu().numpy(), y_ref) <= tol
    y_act = torch.tensor(y_ref, dtype=torch.float32).to(cfg.act_dtype).float().numpy()  # y is an activation
    h_ref = stack.next_hidden(h0.numpy(), y_act, a1.numpy())
    assert oexp.rel_err(hd.cpu().numpy(), h_ref) <= (1e-5 if cfg.act_fmt == "fp32" else 5e-3)
    x_ref = stack.rmsnorm(h_ref)
    assert oexp.rel_err(x1d.float().cpu().numpy(), x_ref) <= (2e-6 if cfg.act_fmt == "fp32" else 2.0 ** -7)
    # routing of layer 1: the logits the device used must match the oracle's up to the rounding of x
    z_ref = routing.router_logits(ow.gate(1), torch.tensor(x_ref).to(cfg.act_dtype).float().numpy())
    z_gpu = np.array(r1.logits[:N], np.float32)
    assert np.abs(z_gpu - z_ref).max() <= (1e-5 if cfg.act_fmt == "fp32" else 3e-2) * np.abs(z_ref).max()
    sel_gpu = list(r1.sel_expert[:K])
    assert sorted(sel_gpu) == sorted(routing.ranking(z_gpu)[:K].tolist())  # empty cache: plain top-K of its own logits
    dec.close()


def run_in_launch_boundary(cfg, T, lam, outputs_every=1, force=True, monkeypatch=None):
    """A coupled stack driven as bench.py drives it - no host waiting for the decision, so that the boundary runs
    in workgroup 0 of the layer's expert launch (reduce_glue_kernel + one expert launch per layer).  Every
    layer-token is checked against the oracle fed with the device's own inputs of that step (its h before the
    step, the y it was handed, its x): h, x, logits, the routing decision incl. slots and misses (tie protocol),
    and, for every outputs_every-th step, y one step later.  Returns (ties, misses)."""
    L, K, N, d = cfg.n_layers, cfg.top_k, cfg.n_experts, cfg.hidden
    if force:
        monkeypatch.setenv("MOE_FUSE_BOUNDARY", "1")  # also without a shared expert (read when the context is created)
    store, dec = build(cfg, lam=lam)
    ow = OracleWeights(cfg)
    routers = [routing.CachePriorRouter(N, K, cfg.capacity, lam, 0, cfg.renormalize) for _ in range(L)]
    a = workloads.ar1_stream(cfg, T)
    a_dev = a.to(DEV)
    h = torch.zeros(d, device=DEV)
    x = torch.zeros(d, dtype=cfg.act_dtype, device=DEV)
    y = torch.zeros(d, dtype=cfg.act_dtype, device=DEV)
    torch.cuda.synchronize()
    assert dec.plan().boundary_in_expert_launch == 1
    ties = misses = step = 0
    y_ref_prev = None  # oracle output of the previous layer-token, from the device's x of that step
    for t in range(T):
        for l in range(L):
            print(f"case in-launch boundary {cfg.name} d={d} token {t} layer {l}", flush=True)
            h_before = h.cpu().numpy().astype(np.float64)
            perturb = 1.0 if l == 0 else stack.PERTURB
            assert dec.stack_route_step(l, h, a_dev[t, l], perturb, x, carry=l > 0, y=y, wait=False) is None
            dec.expert_forward(l, x, None)
            raw = dec.last_route(l)
            dec.compute_stream.synchronize()
            out = route_fields(raw, K)
            ctx = (t, l)
            # y handed out by this boundary = output of the previous layer-token
            if y_ref_prev is not None:
                assert oexp.rel_err(y.float().cpu().numpy(), y_ref_prev) <= 1e-2, ctx
            y_dev = y.float().cpu().numpy().astype(np.float64)
            a_np = a[t, l].double().numpy()
            h_ref = perturb * a_np if l == 0 else stack.next_hidden(h_before, y_dev, a[t, l].numpy())
            assert oexp.rel_err(h.cpu().numpy(), h_ref) <= 1e-5, ctx
            x_ref = stack.rmsnorm(h.cpu().numpy().astype(np.float64))
            x_np = x.float().cpu().numpy()
            assert oexp.rel_err(x_np, x_ref) <= 2.0 ** -7, ctx
            z = routing.router_logits(ow.gate(l), x_np)
            z_gpu = np.array(raw.logits[:N], np.float32)
            assert np.abs(z_gpu - z).max() <= 1e-4 * max(np.abs(z).max(), 1e-3), ctx
            sel, zp, delta = routers[l].select(z)
            if out["sel"] != sel.tolist():
                kth = np.sort(zp)[::-1][K - 1]
                forced = {int(e) for e in np.nonzero(zp > kth + 1e-5)[0]}
                assert np.all(zp[out["sel"]] >= kth - 1e-5) and forced <= set(out["sel"]), (ctx, out["sel"], sel.tolist())
                ties += 1
                sel = np.array(out["sel"])
            ref = routers[l].commit(z, sel, zp, delta)
            assert out["slot"] == ref.slot and out["miss"] == ref.miss and out["evicted"] == ref.evicted, ctx
            misses += sum(ref.miss)
            y_ref_prev = None
            if step % outputs_every == 0:
                y_ref_prev = oexp.moe_output(x_np, [ow.expert(l, int(e)) for e in ref.sel], ref.weight, ow.shared(l))
            step += 1
    for l in range(L):
        s, o = dec.stats(l), routers[l].stats
        assert (s.tokens, s.hits, s.misses, s.evictions) == (o.tokens, o.hits, o.misses, o.evictions)
    print(f"in-launch boundary {cfg.name} d={d}: ties={ties} misses={misses}", flush=True)
    dec.close()
    return ties, misses


@pytest.mark.parametrize("name,hidden,inter", [("c2_qwen_bf16", 2048, 96), ("c2_qwen_bf16", 1024, 64),
                                               ("c2_qwen_bf16", 512, 64), ("c4_dsv2lite_int4", 2048, 128),
                                               ("c4_dsv2lite_int4", 4096, 128), ("c5_mixtral_int8", 4096, 96),
                                               ("c5_mixtral_int8", 1024, 64)])
def test_boundary_inside_the_expert_launch(name, hidden, inter, monkeypatch):
    """Reduced shapes of the three weight formats, every output checked.  Small caches force misses, so the second
    expert launch of a layer is exercised too."""
    base = CONFIGS[name]
    cfg = base.with_(n_layers=3, hidden=hidden, n_experts=12, inter=inter,
                     shared_inter=2 * inter if base.shared_inter else 0, capacity=5, top_k=min(base.top_k, 4),
                     seed=4200 + hidden + inter)
    ties, misses = run_in_launch_boundary(cfg, 16, 0.5, monkeypatch=monkeypatch)
    assert misses > cfg.top_k * cfg.n_layers  # more than the cold misses of the first token


def test_bounded_wait_error_path_and_reset(monkeypatch):
    """Failure handling of the boundary inside the expert launch, forced from the host: with a poll limit of one
    the other workgroups stop waiting before workgroup 0 has routed (no shared expert: the wait comes first).
    Every kernel still ends, the next call that names a layer reports MOE_EHIP, and a reset clears the state."""
    import paper_2412_00099_amd as pkg

    cfg = CONFIGS["c2_qwen_bf16"].with_(n_layers=1, hidden=512, n_experts=12, inter=64, shared_inter=0, capacity=5,
                                        top_k=4, seed=77)
    monkeypatch.setenv("MOE_FUSE_BOUNDARY", "1")
    monkeypatch.setenv("MOE_TAG_SPINS", "1")
    store, dec = build(cfg, lam=0.5)
    assert dec.plan().boundary_in_expert_launch == 1
    a = workloads.ar1_stream(cfg, 1).to(DEV)
    h = torch.zeros(cfg.hidden, device=DEV)
    x = torch.zeros(cfg.hidden, dtype=cfg.act_dtype, device=DEV)
    torch.cuda.synchronize()
    print("case bounded wait: one step with a poll limit of one", flush=True)
    assert dec.stack_route_step(0, h, a[0, 0], 1.0, x, carry=False, y=None, wait=False) is None
    dec.expert_forward(0, x, None)
    dec.compute_stream.synchronize()
    with pytest.raises(pkg.MoEError) as e:
        dec.tables(0)
    assert e.value.code == pkg.MOE_EHIP
    dec.reset()
    assert dec.tables(0).count == 0 and dec.stats(0).tokens == 0
    dec.close()


@pytest.mark.parametrize("ask", ["stats", "tables", "snapshot", "last_route"])
def test_a_wait_that_runs_out_in_a_queued_launch_is_reported(ask, monkeypatch):
    """The host is ahead of the device: the launch whose workgroups stop waiting is still queued when the caller asks.  The
    call that waits for the stream reports it, not the one behind it.  (The stream is held by a kernel of a fixed length.)"""
    import paper_2412_00099_amd as pkg

    cfg = CONFIGS["c2_qwen_bf16"].with_(n_layers=1, hidden=512, n_experts=12, inter=64, shared_inter=0, capacity=5,
                                        top_k=4, seed=77)
    monkeypatch.setenv("MOE_FUSE_BOUNDARY", "1")
    monkeypatch.setenv("MOE_TAG_SPINS", "1")
    store, dec = build(cfg, lam=0.5)
    a = workloads.ar1_stream(cfg, 1).to(DEV)
    h = torch.zeros(cfg.hidden, device=DEV)
    x = torch.zeros(cfg.hidden, dtype=cfg.act_dtype, device=DEV)
    torch.cuda.synchronize()
    print(f"case bounded wait in a queued launch: {ask}", flush=True)
    with torch.cuda.stream(dec.compute_stream):
        torch.cuda._sleep(20_000_000)  # some 10 ms
    dec.stack_route_step(0, h, a[0, 0], 1.0, x, carry=False, y=None, wait=False)
    dec.expert_forward(0, x, None)
    with pytest.raises(pkg.MoEError) as e:
        getattr(dec, ask)(0)
    assert e.value.code == pkg.MOE_EHIP
    dec.reset()
    assert dec.stats(0).tokens == 0
    dec.close()


def test_launch_timing_counts_and_strides():
    """moe_cache_profile: events on every n-th first-pass expert launch; only launches that covered a whole layer
    (no expert missing) are averaged."""
    cfg = CONFIGS["c2_qwen_bf16"].with_(n_layers=2, hidden=512, n_experts=8, inter=64, shared_inter=128, capacity=8,
                                        top_k=2, seed=5)
    store, dec = build(cfg, lam=0.5)
    T = 12
    a = workloads.ar1_stream(cfg, T).to(DEV)
    h = torch.zeros(cfg.hidden, device=DEV)
    x = torch.zeros(cfg.hidden, dtype=cfg.act_dtype, device=DEV)
    torch.cuda.synchronize()

    def run():
        for t in range(T):
            for l in range(cfg.n_layers):
                dec.stack_route_step(l, h, a[t, l], 1.0 if l == 0 else stack.PERTURB, x, carry=l > 0, wait=False)
                dec.expert_forward(l, x, None)
        dec.compute_stream.synchronize()

    print("case launch timing: warm the cache (capacity = all experts)", flush=True)
    run()
    for stride, expect in ((1, T * cfg.n_layers), (5, -(-T * cfg.n_layers // 5))):
        print(f"case launch timing: stride {stride}", flush=True)
        misses_before = dec.stats().misses
        dec.profile(stride, reset=True)
        run()
        avg_us, n = dec.profile(0, reset=True)
        late_misses = dec.stats().misses - misses_before  # a launch with a (late cold) miss is timed but not counted
        assert expect - late_misses <= n <= expect and (n == expect or late_misses > 0)
        assert 0.5 < avg_us < 1000.0
    dec.profile(0, reset=True)
    run()
    assert dec.profile(0, reset=True) == (0.0, 0)
    dec.close()


@pytest.mark.parametrize("weight,act,hidden,inter,shared,N,K,C,mode", [
    ("fp32", "fp32", 1024, 24, 0, 16, 2, 4, 0), ("bf16", "bf16", 2048, 33, 16, 64, 8, 10, 0),
    ("bf16", "bf16", 4096, 20, 0, 9, 4, 6, 0), ("bf16", "fp32", 1024, 40, 8, 60, 5, 60, 1),
    ("int8", "bf16", 1024, 40, 16, 16, 1, 2, 0), ("int8", "bf16", 4096, 24, 0, 8, 2, 4, 2),
    ("int4", "bf16", 2048, 128, 128, 64, 6, 7, 0), ("int4", "fp32", 4096, 128, 0, 12, 3, 3, 0),
    ("bf16", "bf16", 1024, 32, 300, 60, 4, 9, 0)])
def test_routing_in_every_workgroup_equals_the_waiting_path(weight, act, hidden, inter, shared, N, K, C, mode, monkeypatch):
    """A stack driven without waiting (every wavefront of an expert launch routes for itself, the state alternates between
    two copies) against the same stack with a blocking boundary (one workgroup routes ahead of the launch): selections,
    states, outputs and residual streams bit for bit, also with two layers' steps in flight, over a snapshot taken and
    restored, and over a reset."""
    import paper_2412_00099_amd as pkg

    cfg = CONFIGS["c3_olmoe_bf16"].with_(n_layers=2, hidden=hidden, n_experts=N, inter=inter, shared_inter=shared, top_k=K,
                                         capacity=C, weight_fmt=weight, act_fmt=act, seed=5300 + hidden + N)
    print(f"case routing everywhere {weight}/{act} d={hidden} N={N} K={K} C={C} mode={mode}", flush=True)
    monkeypatch.setenv("MOE_ROUTE_EVERYWHERE", "1")  # also where a launch of its own is faster
    kw = dict(lam=0.5, route_mode=mode, max_rank=min(2 * K, N), cumsum_p=0.6, top_j=min(1, K))
    store_a, a = build(cfg, **kw)
    store_b, b = build(cfg, **kw)
    assert not b.plan().boundary_in_expert_launch
    assert b.boundary_form() == pkg.MOE_BOUNDARY_ROUTED_EVERYWHERE
    T, act_dtype = 14, cfg.act_dtype
    stream = workloads.ar1_stream(cfg, T).to(DEV)
    out = []
    for dec, wait in ((a, True), (b, False)):
        h = torch.zeros(2, T, hidden, device=DEV)
        x = torch.zeros(2, hidden, dtype=act_dtype, device=DEV)
        y = torch.zeros(T, hidden, dtype=act_dtype, device=DEV)
        recs = []

        def step(l, t, hh, xx, carry):
            dec.stack_route_step(l, hh, stream[t, l], 1.0 if not carry else 0.5, xx, carry=carry, wait=wait)

        for t in range(T):
            if t == 6:
                dec.restore(1, dec.snapshot(1))
            if t == 9:
                dec.reset()
            if t % 4 == 3:  # both layers routed before either is computed
                step(0, t, h[0, t], x[0], False)
                step(1, t, h[1, t], x[1], False)
                dec.expert_forward(0, x[0], y[t])
                dec.expert_forward(1, x[1], y[t])
            else:
                step(0, t, h[0, t], x[0], False)
                dec.expert_forward(0, x[0], None)
                step(1, t, h[0, t], x[0], True)
                dec.expert_forward(1, x[0], y[t])
            for l in range(2):
                recs.append(bytes(dec.last_route(l))[:-16])
        dec.compute_stream.synchronize()
        out.append((recs, h.cpu(), x.cpu(), y.cpu(), [bytes(dec.tables(l)) for l in range(2)], bytes(dec.stats())))
    for u, v in zip(*out):
        assert torch.equal(u, v) if isinstance(u, torch.Tensor) else u == v
    assert out[0][3].float().abs().max() > 0
    a.close()
    b.close()


@pytest.mark.parametrize("weight,act,hidden", [("fp32", "fp32", 256), ("fp32", "fp32", 512), ("bf16", "bf16", 512)])
def test_routing_in_every_workgroup_small_hidden(weight, act, hidden, monkeypatch):
    """Hidden sizes whose waiting boundary sums the squares of h in another order: x within one rounding of the waiting
    path's, the same decisions, outputs and residual streams to a few roundings."""
    import paper_2412_00099_amd as pkg

    cfg = CONFIGS["c3_olmoe_bf16"].with_(n_layers=1, hidden=hidden, n_experts=16, inter=40, shared_inter=8, top_k=3, capacity=16,
                                         weight_fmt=weight, act_fmt=act, seed=5400 + hidden)
    monkeypatch.setenv("MOE_ROUTE_EVERYWHERE", "1")
    print(f"case routing everywhere, small hidden {weight}/{act} d={hidden}", flush=True)
    store_a, a = build(cfg, lam=0.5)
    store_b, b = build(cfg, lam=0.5)
    assert b.boundary_form() == pkg.MOE_BOUNDARY_ROUTED_EVERYWHERE
    T = 8
    stream = workloads.ar1_stream(cfg, T).to(DEV)
    out = []
    for dec, wait in ((a, True), (b, False)):
        h = torch.zeros(T, hidden, device=DEV)
        x = torch.zeros(T, hidden, dtype=cfg.act_dtype, device=DEV)
        y = torch.zeros_like(x)
        sel = []
        for t in range(T):
            dec.stack_route_step(0, h[t], stream[t, 0], 1.0, x[t], carry=False, wait=wait)
            dec.expert_forward(0, x[t], y[t])
            sel.append(route_fields(dec.last_route(0), cfg.top_k)["sel"])
        dec.compute_stream.synchronize()
        out.append((h.cpu(), x.float().cpu(), y.float().cpu(), sel))
    assert torch.equal(out[0][0], out[1][0]) and out[0][3] == out[1][3]
    # the scale differs by the order of a sum of d squares (a few units of 2^-24); bf16 then rounds to 2^-9
    tol = 1e-6 if act == "fp32" else 2 ** -8
    for u, v in zip(out[0][1:3], out[1][1:3]):
        assert (u - v).abs().max() <= tol * u.abs().max()
    a.close()
    b.close()


@pytest.mark.parametrize("weight,N,K,C,lam,shared", [("bf16", 64, 4, 64, 0.0, 0), ("bf16", 64, 6, 64, 0.0, 16),
                                                    ("bf16", 12, 4, 5, 0.5, 0), ("int8", 12, 3, 12, 0.0, 16),
                                                    ("int4", 64, 2, 64, 0.0, 0)])
def test_routing_in_every_workgroup_without_numbers(weight, N, K, C, lam, shared, monkeypatch):
    """A token that is not a number (its logits fill no places), finite tokens behind it (with lambda = 0 the bias of the
    resident experts is then 0 times no number, so that places stay empty): the expert launch that routes for itself
    takes an empty place for what the record says, as the waiting path does."""
    import paper_2412_00099_amd as pkg

    hidden, inter = (2048, 128) if weight == "int4" else (1024, 24)
    cfg = CONFIGS["c3_olmoe_bf16"].with_(n_layers=1, hidden=hidden, n_experts=N, inter=inter, shared_inter=shared, top_k=K,
                                         capacity=C, weight_fmt=weight, act_fmt="bf16", seed=5600 + N)
    print(f"case routing everywhere without numbers {weight} N={N} K={K} C={C}", flush=True)
    monkeypatch.setenv("MOE_ROUTE_EVERYWHERE", "1")
    monkeypatch.setenv("MOE_FUSE_BOUNDARY", "0")
    initial = [list(range(N))[:C]]
    store_a, a = build(cfg, lam=lam, initial=initial)
    store_b, b = build(cfg, lam=lam, initial=initial)
    assert b.boundary_form() == pkg.MOE_BOUNDARY_ROUTED_EVERYWHERE
    T = 8
    stream = workloads.ar1_stream(cfg, T)[:, 0].contiguous().to(DEV)
    stream[2, 5] = float("nan")
    out = []
    for dec, wait in ((a, True), (b, False)):
        h = torch.zeros(T, hidden, device=DEV)
        x = torch.zeros(T, hidden, dtype=cfg.act_dtype, device=DEV)
        y = torch.zeros_like(x)
        torch.cuda.synchronize()
        recs = []
        for t in range(T):
            dec.stack_route_step(0, h[t], stream[t], 1.0, x[t], carry=False, wait=wait)
            dec.expert_forward(0, x[t], y[t])
            recs.append(route_fields(dec.last_route(0), K))
        dec.compute_stream.synchronize()
        out.append((recs, [v.float().cpu().numpy() for v in (h, x, y)], bytes(dec.stats())))
    for u, v in zip(out[0][0], out[1][0]):
        for key in u:
            assert np.array_equal(u[key], v[key], equal_nan=key in ("weight", "delta", "margin")), (key, u[key], v[key])
    for u, v in zip(out[0][1], out[1][1]):
        assert np.array_equal(u, v, equal_nan=True)
    assert out[0][2] == out[1][2]
    if weight == "bf16":  # (the quantised formats bound the activations on their way to 16-bit floating point)
        assert np.isnan(out[0][1][2][2]).all()
    assert np.isfinite(out[0][1][2][3:]).all()
    a.close()
    b.close()


@pytest.mark.parametrize("sync", ["poll", "event"])
@pytest.mark.parametrize("weight,act,hidden", [("bf16", "bf16", 2048), ("bf16", "bf16", 512), ("fp32", "fp32", 1024),
                                               ("bf16", "bf16", 4096)])
def test_blocking_boundary_returns_with_its_outputs(weight, act, hidden, sync, monkeypatch):
    """A blocking boundary polls for its record while the launch still runs; h, x and the finished y of the layer before
    are complete all the same when it returns: another stream that is not ordered behind compute_stream copies them."""
    if sync == "event":
        monkeypatch.setenv("MOE_HOST_SYNC", "event")
    cfg = CONFIGS["c3_olmoe_bf16"].with_(n_layers=1, hidden=hidden, n_experts=16, inter=24, shared_inter=8, top_k=2, capacity=16,
                                         weight_fmt=weight, act_fmt=act, seed=5700 + hidden)
    print(f"case blocking boundary {weight} d={hidden} {sync}", flush=True)
    store, dec = build(cfg, lam=0.5)
    T = 60
    stream = workloads.ar1_stream(cfg, T)[:, 0].contiguous().to(DEV)
    h = torch.zeros(hidden, device=DEV)
    x = torch.zeros(hidden, dtype=cfg.act_dtype, device=DEV)
    y = torch.zeros_like(x)
    other = torch.cuda.Stream()
    for t in range(T):
        dec.compute_stream.synchronize()  # (the experts have read x)
        x.fill_(float("nan"))
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        dec.stack_route_step(0, h, stream[t], 1.0 if t == 0 else stack.PERTURB, x, carry=t > 0, y=y if t > 0 else None)
        with torch.cuda.stream(other):
            seen = [v.clone() for v in (h, x, y)]
        torch.cuda.synchronize()
        for u, v in zip(seen[: 3 if t > 0 else 2], (h, x, y)):
            assert torch.equal(u, v) and torch.isfinite(u.float()).all(), t
        dec.expert_forward(0, x, None)
    dec.close()


@pytest.mark.parametrize("form", ["MOE_FUSE_BOUNDARY", "MOE_ROUTE_EVERYWHERE"])
@pytest.mark.parametrize("weight,hidden,inter,shared", [("bf16", 2048, 24, 40), ("bf16", 1024, 33, 16), ("int8", 4096, 24, 16),
                                                       ("int4", 2048, 128, 128)])
def test_steps_of_two_layers_in_flight(weight, hidden, inter, shared, form, monkeypatch):
    """Both layers are routed, without waiting, before either is computed - with a residual stream of their own and on
    one that the second step goes on from - in either deferred form of the boundary: as with blocking boundaries."""
    import paper_2412_00099_amd as pkg

    cfg = CONFIGS["c2_qwen_bf16"].with_(n_layers=2, hidden=hidden, n_experts=12, inter=inter, shared_inter=shared, top_k=3,
                                        capacity=5, weight_fmt=weight, act_fmt="bf16", seed=5800 + hidden)
    print(f"case two layers in flight {weight} d={hidden} {form}", flush=True)
    for name in ("MOE_FUSE_BOUNDARY", "MOE_ROUTE_EVERYWHERE"):
        monkeypatch.setenv(name, "1" if name == form else "0")
    T = 10
    stream = workloads.ar1_stream(cfg, T).to(DEV)
    out = []
    for wait in (True, False):
        store, dec = build(cfg, lam=0.5)
        assert dec.boundary_form() == (pkg.MOE_BOUNDARY_IN_FIRST_WORKGROUP if form == "MOE_FUSE_BOUNDARY"
                                       else pkg.MOE_BOUNDARY_ROUTED_EVERYWHERE)
        h = torch.zeros(2, hidden, device=DEV)
        x = torch.zeros(2, hidden, dtype=cfg.act_dtype, device=DEV)
        y = torch.zeros(T, 2, hidden, dtype=cfg.act_dtype, device=DEV)
        torch.cuda.synchronize()
        recs = []
        for t in range(T):
            one = t % 2 == 0  # layer 1 goes on from layer 0's residual stream
            dec.stack_route_step(0, h[0], stream[t, 0], 1.0, x[0], carry=False, wait=wait)
            dec.stack_route_step(1, h[0 if one else 1], stream[t, 1], 0.5 if one else 1.0, x[1], carry=one, wait=wait)
            for l in ((0, 1) if t % 3 else (1, 0)):
                dec.expert_forward(l, x[l], y[t, l])
            recs += [bytes(dec.last_route(l))[:-16] for l in range(2)]
        dec.compute_stream.synchronize()
        out.append((recs, h.cpu(), x.cpu(), y.float().cpu(), [bytes(dec.tables(l)) for l in range(2)], bytes(dec.stats())))
        dec.close()
    for i, (u, v) in enumerate(zip(*out)):
        if i == 3 and form == "MOE_FUSE_BOUNDARY":
            # one workgroup fewer streams records: the order of the sums differs, and with it at most the rounding to bf16
            assert (u - v).abs().max() <= 2 ** -8 * u.abs().max() and u.abs().max() > 0
        else:
            assert torch.equal(u, v) if isinstance(u, torch.Tensor) else u == v


@pytest.mark.parametrize("form", ["MOE_FUSE_BOUNDARY", "MOE_ROUTE_EVERYWHERE", "neither"])
@pytest.mark.parametrize("weight,hidden,inter,shared", [("bf16", 1024, 33, 16), ("int8", 2048, 24, 16), ("int4", 4096, 128, 0)])
def test_tables_counters_and_snapshots_include_the_step_in_flight(weight, hidden, inter, shared, form, monkeypatch):
    """Between a non-blocking boundary and its moe_expert_forward the tables, the counters and a snapshot show the step, in
    whichever form the boundary is run; the experts then compute with the same decision."""
    cfg = CONFIGS["c2_qwen_bf16"].with_(n_layers=2, hidden=hidden, n_experts=12, inter=inter, shared_inter=shared, top_k=3,
                                        capacity=5, weight_fmt=weight, act_fmt="bf16", seed=5900 + hidden)
    print(f"case looking at a step in flight {weight} d={hidden} {form}", flush=True)
    for name in ("MOE_FUSE_BOUNDARY", "MOE_ROUTE_EVERYWHERE"):
        monkeypatch.setenv(name, "1" if name == form else "0")
    T = 8
    stream = workloads.ar1_stream(cfg, T).to(DEV)
    out = []
    for wait in (True, False):
        store, dec = build(cfg, lam=0.5)
        assert dec.boundary_form() == ["neither", "MOE_FUSE_BOUNDARY", "MOE_ROUTE_EVERYWHERE"].index(form)
        h = torch.zeros(hidden, device=DEV)
        x = torch.zeros(hidden, dtype=cfg.act_dtype, device=DEV)
        y = torch.zeros(T, 2, hidden, dtype=cfg.act_dtype, device=DEV)
        torch.cuda.synchronize()
        seen = []
        for t in range(T):
            for l in range(2):
                dec.stack_route_step(l, h, stream[t, l], 1.0 if l == 0 else 0.5, x, carry=l > 0, wait=wait)
                if t % 4 == 0:
                    seen.append(bytes(dec.tables(l)))
                elif t % 4 == 1:
                    seen.append(bytes(dec.stats(l))[:48])  # (bytes_filled: counted once the decision is collected)
                elif t % 4 == 2:
                    seen.append(dec.snapshot(l))
                dec.expert_forward(l, x, y[t, l])
                seen.append(bytes(dec.last_route(l))[:-16])
        seen += [dec.snapshot(l) for l in range(2)] + [bytes(dec.stats())]
        out.append((seen, h.cpu(), y.float().cpu()))
        dec.close()
    assert out[0][0] == out[1][0] and torch.equal(out[0][1], out[1][1])
    # (in one form a workgroup fewer streams records: the rounding of a sum in another order)
    assert (out[0][2] - out[1][2]).abs().max() <= 2 ** -8 * out[0][2].abs().max()


@pytest.mark.parametrize("everywhere", ["0", "1"])
@pytest.mark.parametrize("weight,act,hidden,shared,refused", [("bf16", "bf16", 1024, 64, True), ("int4", "bf16", 2048, 256, True),
                                                            ("bf16", "bf16", 1024, 0, False), ("fp32", "fp32", 1024, 64, False)])
def test_another_x_is_refused_whatever_the_form_of_the_boundary(weight, act, hidden, shared, refused, everywhere, monkeypatch):
    """After a non-blocking boundary moe_expert_forward refuses another vector where the boundary could run inside its launch
    and the shared expert has a third of the records - whether the size rule leaves it there, to every workgroup or to a
    launch of its own - and elsewhere computes with the vector it is given; after a blocking one it always does."""
    import paper_2412_00099_amd as pkg

    monkeypatch.setenv("MOE_ROUTE_EVERYWHERE", everywhere)
    cfg = CONFIGS["c2_qwen_bf16"].with_(n_layers=1, hidden=hidden, n_experts=8, inter=128 if weight == "int4" else 40,
                                        shared_inter=shared, top_k=2, capacity=8, weight_fmt=weight, act_fmt=act, seed=6000)
    store, dec = build(cfg, lam=0.5, initial=[list(range(8))])
    assert dec.boundary_form() == (pkg.MOE_BOUNDARY_ROUTED_EVERYWHERE if everywhere == "1" else pkg.MOE_BOUNDARY_OWN_LAUNCH)
    a = workloads.ar1_stream(cfg, 1).to(DEV)
    h = torch.zeros(hidden, device=DEV)
    x = torch.zeros(hidden, dtype=cfg.act_dtype, device=DEV)
    y, y2 = torch.zeros_like(x), torch.zeros_like(x)
    torch.cuda.synchronize()
    dec.stack_route_step(0, h, a[0, 0], 1.0, x, carry=False)
    other = x.clone()
    torch.cuda.synchronize()
    dec.expert_forward(0, other, y)
    dec.stack_route_step(0, h, a[0, 0], 1.0, x, carry=False, wait=False)
    if refused:
        with pytest.raises(pkg.MoEError) as e:
            dec.expert_forward(0, other, y2)
        assert e.value.code == pkg.MOE_EINVAL
        dec.expert_forward(0, x, y2)
    else:
        dec.expert_forward(0, other, y2)
    dec.compute_stream.synchronize()
    assert torch.equal(y, y2) and y.float().abs().max() > 0
    dec.close()


def test_the_form_of_the_boundary_follows_the_route_mode(monkeypatch):
    """int4 with many experts: the routing is left to every workgroup, except under Cumsum-Threshold; the mode changes from
    token to token, with a step of each form in flight, and everything is as with blocking boundaries."""
    import paper_2412_00099_amd as pkg

    for name in ("MOE_FUSE_BOUNDARY", "MOE_ROUTE_EVERYWHERE"):
        monkeypatch.delenv(name, raising=False)
    cfg = CONFIGS["c4_dsv2lite_int4"].with_(n_layers=1, n_experts=40, inter=1152, shared_inter=0, top_k=4, capacity=9, seed=6100)
    print("case boundary form by route mode", flush=True)
    modes = [(pkg.MOE_ROUTE_CACHE_PRIOR, 0, 0.0, pkg.MOE_BOUNDARY_ROUTED_EVERYWHERE),
             (pkg.MOE_ROUTE_CUMSUM, 0, 0.6, pkg.MOE_BOUNDARY_OWN_LAUNCH),
             (pkg.MOE_ROUTE_MAX_RANK, 8, 0.0, pkg.MOE_BOUNDARY_ROUTED_EVERYWHERE)]
    T = 9
    stream = workloads.ar1_stream(cfg, T)[:, 0].contiguous().to(DEV)
    out = []
    for wait in (True, False):
        store, dec = build(cfg, lam=0.5)
        h = torch.zeros(cfg.hidden, device=DEV)
        x = torch.zeros(cfg.hidden, dtype=cfg.act_dtype, device=DEV)
        y = torch.zeros(T, cfg.hidden, dtype=cfg.act_dtype, device=DEV)
        torch.cuda.synchronize()
        recs = []
        for t in range(T):
            mode, max_rank, p, form = modes[t * t % 3 if t % 2 else t % 3]
            dec.set_baseline(mode, max_rank, p)
            assert dec.boundary_form() == form
            dec.stack_route_step(0, h, stream[t], 1.0 if t == 0 else 0.5, x, carry=t > 0, wait=wait)
            dec.set_baseline(*modes[(t + 1) % 3][:3])  # (the step in flight keeps its mode)
            dec.expert_forward(0, x, y[t])
            recs.append(bytes(dec.last_route(0))[:-16])
        dec.compute_stream.synchronize()
        out.append((recs, h.cpu(), y.cpu(), bytes(dec.tables(0)), bytes(dec.stats())))
        dec.close()
    for u, v in zip(*out):
        assert torch.equal(u, v) if isinstance(u, torch.Tensor) else u == v


@pytest.mark.parametrize("weight,hidden,inter,shared", [("bf16", 2048, 24, 72), ("bf16", 512, 64, 0), ("int8", 4096, 24, 16),
                                                       ("int4", 2048, 128, 128)])
def test_contexts_in_flight_together(weight, hidden, inter, shared, monkeypatch):
    """The boundary in the first workgroup of the expert launch has the others wait: only one context at a time may have such
    launches on the device.  A decoder whose stream is held up has the turn; a second one (which would give up at its first
    poll) goes through all of its tokens meanwhile, with the same bits as alone, misses among them; then the first one does."""
    import paper_2412_00099_amd as pkg

    cfg = CONFIGS["c2_qwen_bf16"].with_(n_layers=2, hidden=hidden, n_experts=12, inter=inter, shared_inter=shared, top_k=3,
                                        capacity=5, weight_fmt=weight, act_fmt="bf16", seed=6200 + hidden)
    print(f"case contexts in flight together {weight} d={hidden}", flush=True)
    monkeypatch.setenv("MOE_FUSE_BOUNDARY", "1")
    T = 8
    stream = workloads.ar1_stream(cfg, T).to(DEV)

    def run(dec, bufs):
        h, x, y = bufs
        for t in range(T):
            for l in range(2):
                dec.stack_route_step(l, h[t], stream[t, l], 1.0 if l == 0 else 0.5, x[t, l], carry=l > 0, wait=False)
                dec.expert_forward(l, x[t, l], y[t] if l else None)

    def buffers():
        return (torch.zeros(T, hidden, device=DEV), torch.zeros(T, 2, hidden, dtype=cfg.act_dtype, device=DEV),
                torch.zeros(T, hidden, dtype=cfg.act_dtype, device=DEV))

    def result(dec, bufs):
        dec.compute_stream.synchronize()
        return [v.cpu() for v in bufs], [bytes(dec.tables(l)) for l in range(2)], bytes(dec.stats())

    def same(u, v):
        return all(torch.equal(p, q) for p, q in zip(u[0], v[0])) and u[1:] == v[1:]

    _, alone = build(cfg, lam=0.5)
    assert alone.boundary_form() == pkg.MOE_BOUNDARY_IN_FIRST_WORKGROUP
    bufs = [buffers() for _ in range(4)]
    torch.cuda.synchronize()
    run(alone, bufs[0])
    ref = result(alone, bufs[0])
    alone.close()
    assert alone.ctx is None and ref[0][2].float().abs().max() > 0

    _, a = build(cfg, lam=0.5)
    monkeypatch.setenv("MOE_TAG_SPINS", "1")
    _, b = build(cfg, lam=0.5)
    torch.cuda.synchronize()
    held = torch.cuda.Event()
    with torch.cuda.stream(a.compute_stream):
        torch.cuda._sleep(400_000_000)  # a good part of a second
        held.record()
    run(a, bufs[1])
    run(b, bufs[2])
    assert not held.query()  # (all of b's steps were enqueued while none of a's were decided)
    assert same(result(b, bufs[2]), ref)
    assert same(result(a, bufs[1]), ref)
    b.close()
    # ... and once a's decisions are known the turn is free again
    monkeypatch.delenv("MOE_TAG_SPINS")
    _, c = build(cfg, lam=0.5)
    torch.cuda.synchronize()
    run(c, bufs[3])
    assert same(result(c, bufs[3]), ref)
    a.close()
    c.close()

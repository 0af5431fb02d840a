"""The same inputs give the same bits from version to version: digests of fp32 outputs of the allocation-free entry point, for
every weight format, hidden size and enough records that a wavefront walks several (whichever copy of its loop adds a record,
the sums are rounded alike); and routed steps, whose kernels are compiled apart, give the bits of that entry point.  Parity unpinned: the digests are those of an earlier build of this library, whose outputs the other
tests hold against the oracle; they belong to 256 compute units, which is what the records are split over."""
import ctypes as C
import hashlib

import numpy as np
import pytest
import torch

import paper_2412_00099_amd as moe

DEV = "cuda:0"
# (weights, hidden, inter, shared, top_k): sha256 of y, the first 16 digits
BITS = {
    ("fp32", 256, 700, 90, 3): "52491806b595ddbc",
    ("fp32", 2048, 1500, 0, 4): "70270b7439bb801c",
    ("bf16", 512, 2000, 300, 4): "03ca8f093d2a9545",
    ("bf16", 1024, 1024, 0, 8): "1886229733a1e5d9",
    ("bf16", 2048, 1408, 2000, 4): "9d533ece33a85bb1",
    ("bf16", 4096, 900, 0, 4): "a415da9aeef33c54",
    ("int8", 1024, 2000, 0, 5): "ddc9af1646c2619f",
    ("int8", 2048, 1000, 0, 6): "fa5f42b174e48c9f",
    ("int8", 2048, 1408, 1600, 6): "c4ca738b36d13bf5",
    ("int8", 4096, 2048, 0, 2): "b100349ebb08bcf2",
    ("int4", 2048, 1408, 2816, 6): "8dcb4f9c1a7aac62",
    ("int4", 2048, 1024, 0, 3): "3dbdd92b724f49ed",
    ("int4", 4096, 1280, 256, 4): "66d00e4db38b8bdc",
}


def _blob(fmt, hidden, inter, rng):
    def matrix(rows, cols):
        if fmt == "fp32":
            return rng.standard_normal((rows, cols), dtype=np.float32) * np.float32(0.02), None
        if fmt == "bf16":
            bits = (rng.standard_normal((rows, cols), dtype=np.float32) * np.float32(0.02)).view(np.uint32) >> 16
            return bits.astype(np.uint16).view(np.int16), None
        if fmt == "int8":
            return rng.integers(-127, 128, (rows, cols), dtype=np.int8), (rng.random(rows, dtype=np.float32) * 4e-4).astype(np.float16)
        return (rng.integers(0, 256, (rows, cols // 2), dtype=np.uint8),
                (rng.random((rows, cols // 128), dtype=np.float32) * 6e-3).astype(np.float16))

    parts = [matrix(inter, hidden), matrix(inter, hidden), matrix(hidden, inter)]
    keep = [(torch.from_numpy(w).to(DEV), None if s is None else torch.from_numpy(s).to(DEV)) for w, s in parts]
    blob = torch.zeros(moe.moe_blob_bytes(moe.WEIGHT_FMT[fmt], hidden, inter), dtype=torch.uint8, device=DEV)
    ptr = lambda t: None if t is None else C.c_void_p(t.data_ptr())  # noqa: E731
    torch.cuda.synchronize()
    moe.moe_pack_expert(moe.WEIGHT_FMT[fmt], hidden, inter, *[ptr(w) for w, _ in keep], *[ptr(s) for _, s in keep], ptr(blob),
                        C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    return blob


def digest(fmt, hidden, inter, shared, top_k):
    rng = np.random.default_rng([hidden, inter, shared, top_k])
    pool = torch.stack([_blob(fmt, hidden, inter, rng) for _ in range(top_k)])
    shared_blob = _blob(fmt, hidden, shared, rng) if shared else None
    x = torch.from_numpy(rng.standard_normal(hidden, dtype=np.float32)).to(DEV)
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    moe.moe_expert_forward_static(moe.WEIGHT_FMT[fmt], moe.ACT_FMT["fp32"], hidden, inter, shared, top_k,
                                  C.c_void_p(pool.data_ptr()), top_k, None if not shared else C.c_void_p(shared_blob.data_ptr()),
                                  list(range(top_k)), [float(w) for w in rng.random(top_k, dtype=np.float32)],
                                  C.c_void_p(x.data_ptr()), C.c_void_p(y.data_ptr()),
                                  C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    out = y.cpu().numpy()
    assert np.isfinite(out).all() and np.abs(out).max() > 0
    return hashlib.sha256(out.tobytes()).hexdigest()[:16]


@pytest.mark.gpu
@pytest.mark.parametrize("case", sorted(BITS))
def test_bits(case):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the digests are for 256 compute units")
    print("case bits", case, flush=True)
    assert digest(*case) == BITS[case]


@pytest.mark.gpu
@pytest.mark.parametrize("way", ["waited for", "routed ahead", "routed everywhere"])
@pytest.mark.parametrize("case", [c for c in sorted(BITS) if c[1] >= 1024])
def test_routed_steps_give_the_same_bits(case, way, monkeypatch):
    fmt, hidden, inter, shared, top_k = case
    print("case routed bits", case, way, flush=True)
    monkeypatch.setenv("MOE_ROUTE_EVERYWHERE", "1" if way == "routed everywhere" else "0")
    rng, n = np.random.default_rng([hidden, inter, shared, top_k, 1]), top_k + 1
    store = moe.ExpertStore(n_layers=1, hidden=hidden, n_experts=n, inter=inter, shared_inter=shared, capacity=n, weight_fmt=fmt,
                            act_fmt="fp32", device=DEV)
    for e in range(n):
        store.host[0, e].copy_(_blob(fmt, hidden, inter, rng))
    if shared:
        store.shared[0].copy_(_blob(fmt, hidden, shared, rng))
    store.put_gate(0, torch.from_numpy(rng.standard_normal((n, hidden), dtype=np.float32) * np.float32(0.02)))
    x = torch.from_numpy(rng.standard_normal(hidden, dtype=np.float32)).to(DEV)
    y, y_static = torch.zeros_like(x), torch.zeros_like(x)
    dec = moe.MoEDecoder(store, top_k=top_k, lam=0.0, initial=[list(range(n))])
    dec.route_step(0, x=x, wait=way == "waited for")
    dec.expert_forward(0, x, y)
    rec = dec.last_route(0)
    moe.moe_expert_forward_static(moe.WEIGHT_FMT[fmt], moe.ACT_FMT["fp32"], hidden, inter, shared, top_k,
                                  C.c_void_p(store.pools[0].data_ptr()), n, C.c_void_p(store.shared[0].data_ptr()) if shared else None,
                                  list(rec.sel_slot)[:top_k], list(rec.sel_weight)[:top_k], C.c_void_p(x.data_ptr()),
                                  C.c_void_p(y_static.data_ptr()), C.c_void_p(dec.compute_stream.cuda_stream))
    torch.cuda.synchronize()
    dec.close()
    assert not any(list(rec.miss)[:top_k]) and float(y.abs().max()) > 0
    assert torch.equal(y, y_static)

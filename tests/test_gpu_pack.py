"""moe_pack_expert against the record layout written out with plain tensor operations: byte for byte, every format, at
the edges of the packers' tiles and with inputs that are not 16-byte aligned (views into a larger tensor)."""
import ctypes as C

import pytest
import torch

from _gpu_common import DEV

pytestmark = pytest.mark.gpu


def as_bytes(t):
    return t.contiguous().view(torch.uint8).flatten()


def layout(fmt, d, I, w, s):
    """record i = gate row i | up row i | column i of down (int4: | its scale pairs, padded to 128 bytes), then the tail."""
    gate, up, down = (t.cpu() for t in w)
    if fmt == "int8":
        gate, up, down = (t.view(torch.uint8) ^ 0x80 for t in (gate, up, down))
    if fmt == "int4":
        q = torch.stack((down & 15, down >> 4), 2).reshape(d, I)
        column = (q.t()[:, 0::2] | (q.t()[:, 1::2] << 4)).contiguous()
        pairs = torch.stack((s[0].cpu(), s[1].cpu()), 2).contiguous().view(torch.uint8).reshape(I, -1)
        pad = torch.zeros(I, -pairs.shape[1] % 128, dtype=torch.uint8)
        records = torch.cat((gate, up, column, pairs, pad), 1)
        return torch.cat((records.flatten(), as_bytes(s[2].cpu().t())))
    records = torch.stack((gate, up, down.t()), 1)
    if fmt == "int8":
        return torch.cat([as_bytes(records)] + [as_bytes(t.cpu()) for t in s])
    return as_bytes(records)


def shifted(t, offset):
    """The same values in memory that starts `offset` elements into an allocation."""
    if t is None or offset == 0:
        return t
    flat = torch.empty(t.numel() + offset, dtype=t.dtype, device=t.device)
    flat[offset:].copy_(t.flatten())
    return flat[offset:].view(t.shape)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("fmt,d,I", [("fp32", 256, 1), ("fp32", 512, 33), ("fp32", 1024, 64), ("bf16", 512, 1), ("bf16", 512, 63),
                                     ("bf16", 2048, 72), ("bf16", 1024, 129), ("int8", 1024, 8), ("int8", 2048, 136),
                                     ("int8", 1024, 72), ("int4", 2048, 128), ("int4", 4096, 256)])
def test_pack_layout(fmt, d, I, offset):
    import paper_2412_00099_amd as pkg

    print(f"case pack {fmt} d={d} I={I} offset={offset}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(d + I)
    if fmt in ("fp32", "bf16"):
        dtype = torch.float32 if fmt == "fp32" else torch.bfloat16
        w = [torch.randn(r, c, generator=g, device=DEV).to(dtype) for r, c in ((I, d), (I, d), (d, I))]
        s = [None] * 3
    elif fmt == "int8":
        w = [torch.randint(-128, 128, rc, generator=g, device=DEV, dtype=torch.int8) for rc in ((I, d), (I, d), (d, I))]
        s = [torch.rand(n, generator=g, device=DEV).half() for n in (I, I, d)]
    else:
        w = [torch.randint(0, 256, rc, generator=g, device=DEV, dtype=torch.uint8) for rc in ((I, d // 2), (I, d // 2), (d, I // 2))]
        s = [torch.rand(*rc, generator=g, device=DEV).half() for rc in ((I, d // 128), (I, d // 128), (d, I // 128))]
    n = pkg.moe_blob_bytes(pkg.WEIGHT_FMT[fmt], d, I)
    blob = torch.zeros(n, dtype=torch.uint8, device=DEV)
    w_in, s_in = [shifted(t, offset) for t in w], [shifted(t, offset) for t in s]
    ptr = lambda t: None if t is None else C.c_void_p(t.data_ptr())  # noqa: E731
    torch.cuda.synchronize()
    pkg.moe_pack_expert(pkg.WEIGHT_FMT[fmt], d, I, *[ptr(t) for t in w_in], *[ptr(t) for t in s_in], ptr(blob),
                        C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    ref = layout(fmt, d, I, w, s)
    assert torch.equal(blob.cpu()[:ref.numel()], ref)

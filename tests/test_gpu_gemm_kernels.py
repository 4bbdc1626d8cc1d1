"""Every decoded-operand GEMM kernel on operands that hold every block-scale
code and nibble, at the edges of its tiles: 256 x 256 tiles with even, odd and
ragged stage counts, one and several tiles per workgroup, split and small
leftover tiles, both epilogues; the streaming kernel; blocks of 32 and E4M3
scales through them.  Every output is compared in binary64 to the fp32
accumulation bound of tests/gpu_util.gemm_check, C lies inside a guarded
buffer, and the bf16 output is the rounded fp32 one.

Which kernels a size runs on is a choice by modelled time, so the names given
per case are checked on the host (test_host_launches.py).  The staged and the
general kernel, which serve operands past 2^31 bytes, are in
test_gpu_large.py, the small tiles by themselves in test_gpu_gemm_mid.py."""

import numpy as np
import pytest
import torch

import paper_2609_02846_amd as ue
from oracle import quantize as oq
from tests.gpu_util import f32_scalar_dev, say, u8_to_dev

pytestmark = pytest.mark.gpu

# (layout, M, N, K, fmt, block), kernels
CASES = [
    # 256 x 256 tiles, one per CU: vector and per-element epilogue
    (("nt", 4096, 4096, 512, "ue5m3", 16), ["large"]),
    (("nn", 4090, 4080, 512, "e4m3", 16), ["large"]),
    (("tn", 4089, 4094, 512, "ue5m3", 16), ["large masked"]),
    # odd stage counts: one item per workgroup, two rounds
    (("nn", 4090, 8176, 768, "ue5m3", 16), ["large"]),
    (("tn", 4094, 8190, 768, "e4m3", 16), ["large masked"]),
    # persistent: two whole tiles of some workgroups
    (("nt", 4090, 7920, 512, "ue5m3", 16), ["large"]),
    (("tn", 4087, 7922, 512, "ue5m3", 16), ["large masked"]),
    # a split last wave, even and odd stage counts
    (("nt", 4090, 4352, 1024, "ue5m3", 16), ["large", "sum"]),
    (("tn", 4222, 4398, 1280, "ue5m3", 16), ["large masked", "sum"]),
    # K % 256 != 0: odd and even stage counts, small leftover tiles
    (("nt", 4096, 4096, 2064, "e4m3", 16), ["large ragged K"]),
    (("tn", 4089, 4094, 2000, "ue5m3", 16), ["large masked ragged K"]),
    (("nn", 4090, 4592, 2128, "ue5m3", 16), ["large ragged K", "64x128 k2"]),
    # blocks of 32: code rows whose length is a multiple of four codes and not
    (("nt", 4096, 4096, 512, "e4m3", 32), ["codes", "large"]),
    (("tn", 4089, 4094, 2016, "ue5m3", 32), ["codes", "large masked ragged K"]),
    (("nn", 300, 288, 480, "ue5m3", 32), ["codes", "64x64"]),
    # the streaming kernel: whole and partial steps
    (("nt", 64, 4096, 1152, "ue5m3", 16), ["stream 4x2 w4"]),
    (("tn", 13, 4103, 1168, "e4m3", 16), ["stream 1x1 w4"]),
    (("nn", 32, 8192, 544, "ue5m3", 32), ["codes", "stream 2x2 w4"]),
]
LAST_CODE = {"ue5m3": 0xF7, "e4m3": 0x7E}


def _operand(rng, rows, K, tiled, fmt, block, codes=None):
    """Raw payload and scale codes (every finite code of the format, shuffled,
    or those of ``codes``) and the decoded matrix, on the GPU."""
    p = rng.integers(0, 256, (rows, K // 2), dtype=np.uint8)
    shape = (rows // block if tiled else rows, K // block)
    lo, hi = (0, LAST_CODE[fmt] + 1) if codes is None else codes
    s = lo + np.arange(shape[0] * shape[1]) % (hi - lo)
    rng.shuffle(s)
    s = s.reshape(shape).astype(np.uint8)
    dec = (oq.decoded_2d(p, s, fmt=fmt, tile=block) if tiled else oq.decoded_1d(p, s, 1, fmt=fmt, block=block))
    return u8_to_dev(p), u8_to_dev(s), torch.from_numpy(np.ascontiguousarray(dec, np.float64)).cuda()


@pytest.mark.parametrize("layout,M,N,K,fmt,block", [c for c, _ in CASES])
def test_every_code_on_every_kernel(layout, M, N, K, fmt, block):
    say("gemm kernels", layout, M, N, K, fmt, block)
    rng = np.random.default_rng(M + K)
    a, sa, A = _operand(rng, M, K, False, fmt, block)
    b, sb, B = _operand(rng, N, K, layout != "tn", fmt, block)
    da, db = np.float32(1.0 / 2688.0), np.float32(0.75 / 2688.0)
    al = float(np.float32(da * db))
    want, bound = al * (A @ B.T), al * K * 2.0 ** -23 * (A.abs() @ B.abs().T)
    args = (layout, M, N, K, a, sa, f32_scalar_dev(da), b, sb, f32_scalar_dev(db))
    kw = dict(fmt=fmt, block=block)
    pre, post = 4096, ((M + 255) // 256 * 256 - M + 256) * N
    buf = torch.full((pre + M * N + post,), float("nan"), device="cuda")
    c = buf[pre:pre + M * N].view(M, N)
    ue.gemm(*args, out=c, **kw)
    torch.cuda.synchronize()
    err = (c.double() - want).abs()
    assert bool((err <= bound + 2.0 ** -23 * want.abs()).all()), f"worst {float((err / bound.clamp_min(1e-300)).max())}"
    assert bool(buf[:pre].isnan().all()) and bool(buf[pre + M * N:].isnan().all()), "written outside C"
    buf16 = torch.full((pre + M * N + post,), float("nan"), dtype=torch.bfloat16, device="cuda")
    c16 = buf16[pre:pre + M * N].view(M, N)
    ue.gemm(*args, out=c16, **kw)
    torch.cuda.synchronize()
    assert torch.equal(c16, c.to(torch.bfloat16))
    assert bool(buf16[:pre].isnan().all()) and bool(buf16[pre + M * N:].isnan().all()), "written outside C"
    if fmt == "ue5m3" and block == 16:
        na = torch.empty(M, N, device="cuda")
        ue.gemm_noalloc(*args, na)
        torch.cuda.synchronize()
        assert torch.equal(na, c)


# the kernels whose decode and accumulation differ
SMALLEST = [(("nt", 4096, 4096, 512), ["large"]), (("nt", 4096, 4096, 2064), ["large ragged K"]),
            (("nt", 256, 256, 512), ["64x64"]), (("nt", 64, 2048, 1040), ["stream 4x1 w4"])]


@pytest.mark.parametrize("fmt", ["ue5m3", "e4m3"])
@pytest.mark.parametrize("layout,M,N,K", [c for c, _ in SMALLEST])
def test_smallest_codes_are_exact(layout, M, N, K, fmt):
    """Only the subnormal codes and the smallest normal one: decoded values
    reach 2^-21 on the matrix cores' fp16 operands.  Products are multiples of
    2^-36 (E4M3: 2^-20) and their sums stay below 2^24 of it, so outputs equal
    the exact sums."""
    say("gemm smallest codes", layout, M, N, K, fmt)
    rng = np.random.default_rng(K)
    a, sa, A = _operand(rng, M, K, False, fmt, 16, (1, 9))
    b, sb, B = _operand(rng, N, K, True, fmt, 16, (1, 9))
    want = A @ B.T
    unit = 2.0 ** -36 if fmt == "ue5m3" else 2.0 ** -20
    assert float(want.abs().max()) < 2.0 ** 24 * unit
    one = f32_scalar_dev(1.0)
    c = ue.gemm(layout, M, N, K, a, sa, one, b, sb, one, fmt=fmt)
    torch.cuda.synchronize()
    assert torch.equal(c.double(), want)

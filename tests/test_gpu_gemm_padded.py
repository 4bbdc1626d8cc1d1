"""Large decoded-operand products whose K is not a multiple of 256 (256 x 256
tiles whose last stage runs past the rows' end): odd and even stage counts,
K / 16 odd (the last row ends inside a 16-byte chunk), leftover tiles in every
smaller size, ragged M and N, both epilogues and scale layouts, the
allocation-free call, and a capture on a stream without workspaces, which
has to run the same kernels.  Raw codes; reference in float64 with the fp32
accumulation bound.  The kernels named per case are checked on the host
(test_host_launches.py)."""

import pytest
import torch

import paper_2609_02846_amd as ue
from tests.gpu_util import f32_scalar_dev, say

pytestmark = pytest.mark.gpu


def _operand(rows, K, tiled, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    p = torch.randint(0, 256, (rows, K // 2), dtype=torch.uint8, device="cuda", generator=g)
    s = torch.randint(0x60, 0x90, (rows // 16 if tiled else rows, K // 16), dtype=torch.uint8, device="cuda",
                      generator=g)
    mag = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6], dtype=torch.float64, device="cuda")
    nib = torch.stack([p & 15, p >> 4], 2).reshape(rows, K).long()
    sv = torch.exp2((s >> 3).double() - 15) * (1 + (s & 7).double() / 8)
    sv = sv.repeat_interleave(16, 1)
    return p, s, torch.cat([mag, -mag])[nib] * (sv.repeat_interleave(16, 0) if tiled else sv)


# (layout, M, N, K), kernels
CASES = [
    (("nt", 4096, 4096, 4080), ["large ragged K"]),                                # 16 stages
    (("tn", 4096, 4096, 2064), ["large ragged K"]),                                # 9 stages
    (("tn", 4089, 4094, 2064), ["large masked ragged K"]),
    (("tn", 4097, 4096, 4048), ["large ragged K", "64x64 k2"]),                    # 16 tiles left over
    (("nn", 4090, 4592, 4080), ["large ragged K", "64x128 k2"]),                   # 32
    (("tn", 4222, 4397, 2064), ["large masked ragged K", "128x128 k2"]),           # 50
    (("nn", 4100, 4400, 2064), ["large ragged K", "128x128 k2"]),                  # 50
    (("tn", 4093, 6141, 4048), ["large masked ragged K", "128x128"]),              # 128
    (("tn", 8190, 4099, 2064), ["large masked ragged K", "64x128 k2"]),            # two whole waves and 32
]


@pytest.mark.parametrize("layout,M,N,K", [c for c, _ in CASES])
def test_padded_scale_codes(layout, M, N, K):
    say("padded gemm", layout, M, N, K)
    a, sa, A = _operand(M, K, False, 51)
    b, sb, B = _operand(N, K, layout != "tn", 52)
    one = f32_scalar_dev(1.0)
    want = A @ B.T
    bound = K * 2.0 ** -23 * (A.abs() @ B.abs().T) + 2.0 ** -23 * want.abs()
    ok = lambda c: bool(((c.double() - want).abs() <= bound).all())  # noqa: E731
    args = (layout, M, N, K, a, sa, one, b, sb, one)
    guard = torch.full((M * N + 4096,), 7.25, device="cuda")
    c = ue.gemm(*args, out=guard[:M * N].view(M, N))
    torch.cuda.synchronize()
    assert ok(c) and bool((guard[M * N:] == 7.25).all())
    assert torch.equal(ue.gemm(*args, out_dtype=torch.bfloat16), c.to(torch.bfloat16))
    na = torch.empty(M, N, device="cuda")
    ue.gemm_noalloc(*args, na)
    torch.cuda.synchronize()
    assert torch.equal(na, c)
    # a capturing stream without workspaces: the same kernels and bits
    out = torch.zeros(M, N, device="cuda")
    st, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=st):
        ue.gemm(*args, out=out)
    for _ in range(2):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, c)

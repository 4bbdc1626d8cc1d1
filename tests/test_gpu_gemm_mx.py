"""E8M0 GEMM on the scaled FP4 instructions at the edges of its walk: one, odd
and even numbers of 256-k stages (scale codes come in pairs of stages), one and
several tiles per workgroup, split tails with odd stage ranges, ragged M and N,
both epilogues and output types.  Operands are raw codes; the expected sums are
exact in binary64 (products of E2M1 values and powers of two within 2^-8 ..
2^8 over at most 1536 terms) and in binary32, so outputs are equal."""

import pytest
import torch

import paper_2609_02846_amd as ue
from tests.gpu_util import f32_scalar_dev, say

pytestmark = pytest.mark.gpu


def _operand(rows, K, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    p = torch.randint(0, 256, (rows, K // 2), dtype=torch.uint8, device="cuda", generator=g)
    s = torch.randint(125, 129, (rows, K // 32), dtype=torch.uint8, device="cuda", generator=g)
    mag = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6], dtype=torch.float64, device="cuda")
    table = torch.cat([mag, -mag])
    nib = torch.stack([p & 15, p >> 4], 2).reshape(rows, K).long()
    return p, s, table[nib] * torch.exp2(s.double() - 127).repeat_interleave(32, 1)


# (M, N, K): 17 x 17 = 289 tiles leave a last wave of 33 (split), 34 x 17 = 578
# two whole waves and 66 split tiles; N % 8 and N % 4 choose the epilogue
@pytest.mark.parametrize("M,N,K", [(256, 256, 256), (300, 520, 768), (77, 100, 1280), (4300, 4352, 768),
                                   (4352, 4350, 512), (8700, 4104, 1280)])
def test_stage_and_item_edges(M, N, K):
    say("mx gemm", M, N, K)
    a, sa, A = _operand(M, K, 41)
    b, sb, B = _operand(N, K, 42)
    one = f32_scalar_dev(1.0)
    want = (A @ B.T).float()
    for dt in (torch.float32, torch.bfloat16):
        guard = torch.full((M * N + 4096,), 7.25, dtype=dt, device="cuda")
        c = ue.gemm("nt", M, N, K, a, sa, one, b, sb, one, out=guard[:M * N].view(M, N), fmt="e8m0")
        torch.cuda.synchronize()
        assert torch.equal(c, want.to(dt)), f"{M}x{N}x{K} {dt}"
        assert bool((guard[M * N:] == 7.25).all())

"""Decoded-operand GEMM with few output rows (M <= 64, the streaming kernel):
every group count, both weight-row widths, short and long K, K with a partial
step, the last M and N, both output types and both scale layouts, against the
oracle to the GEMM bar."""

import pytest
import torch

import paper_2609_02846_amd as ue
import synthetic
from oracle import gemm as ogemm
from oracle import quantize as oq
from oracle import scaling as osc
from tests.gpu_util import f32_scalar_dev, gemm_check, host, say, u8_to_dev

pytestmark = pytest.mark.gpu

# (layout, M, N, K): N below and above both width limits, K % 128 != 0, K past
# the wave-count limit, single rows and the last row count of each group
CASES = [("nt", 1, 256, 128), ("nt", 16, 4096, 16), ("nt", 17, 48, 4112), ("tn", 33, 4103, 144),
         ("nn", 32, 8192, 272), ("tn", 64, 8195, 256), ("nt", 64, 4096, 1040), ("tn", 5, 37, 4224)]


@pytest.mark.parametrize("layout,M,N,K", CASES)
def test_few_rows(layout, M, N, K):
    say("skinny gemm", layout, M, N, K)
    tiled = layout != "tn"
    x = synthetic.activation(11, M, K, 0.01, 50.0)
    w = synthetic.weight(12, N, K)
    xq = oq.quantize_1d(x, 1, osc.amax(x))
    if tiled:
        wq = oq.quantize_2d(w, osc.amax(w))
        b, bs, db = wq[0], wq[1], wq[3]
        W = oq.decoded_2d(b, bs)
    else:
        b, bs, db = oq.quantize_1d(w, 1, osc.amax(w))[:3]
        W = oq.decoded_1d(b, bs, 1)
    X = oq.decoded_1d(xq[0], xq[1], 1)
    al = ogemm.alpha(xq[2], db)
    args = (u8_to_dev(xq[0]), u8_to_dev(xq[1]), f32_scalar_dev(xq[2]), u8_to_dev(b), u8_to_dev(bs),
            f32_scalar_dev(db))
    guard = torch.full((M * N + 64,), 7.25, dtype=torch.float32, device="cuda")
    out = guard[:M * N].view(M, N)
    ue.gemm(layout, M, N, K, *args, out=out)
    torch.cuda.synchronize()
    gemm_check(host(out), ogemm.fprop(X, W, al), al, ogemm.abs_product(X, W), K, f"{layout} {M}x{N}x{K}")
    assert bool((guard[M * N:] == 7.25).all())
    b16 = ue.gemm(layout, M, N, K, *args, out_dtype=torch.bfloat16)
    na = torch.empty(M, N, device="cuda")
    ue.gemm_noalloc(layout, M, N, K, *args, na)
    torch.cuda.synchronize()
    assert torch.equal(b16, out.to(torch.bfloat16))
    assert torch.equal(na, out)

"""Decoded-operand GEMM with few output rows (M <= 64): the streaming kernel at
every group count, both weight-row widths, short and long K, K with a partial
step, the last M and N, and both sides of the lines beyond which more than 32
rows run in small tiles; both output types and scale layouts, against the
oracle to the GEMM bar.  The kernels named per case are checked on the host
(test_host_launches.py)."""

import pytest
import torch

import paper_2609_02846_amd as ue
import synthetic
from oracle import gemm as ogemm
from oracle import quantize as oq
from oracle import scaling as osc
from tests.gpu_util import f32_scalar_dev, gemm_check, host, say, u8_to_dev

pytestmark = pytest.mark.gpu

# (layout, M, N, K), kernel: N below and above both width limits, K % 128 != 0,
# K past the wave-count limit, single rows and the last row count of each group
CASES = [
    (("nt", 1, 256, 128), "stream 1x1 w4"), (("nt", 16, 4096, 16), "stream 1x1 w4"),
    (("tn", 5, 37, 4224), "stream 1x1 w8"), (("tn", 16, 8195, 144), "stream 1x2 w4"),
    (("nt", 17, 48, 4112), "stream 2x1 w8"), (("nt", 32, 1040, 4096), "stream 2x1 w4"),
    (("nn", 32, 8192, 272), "stream 2x2 w4"), (("tn", 29, 8209, 2048), "stream 2x2 w4"),
    (("nt", 64, 2048, 1040), "stream 4x1 w4"), (("tn", 33, 4095, 4240), "stream 4x1 w8"),
    (("nt", 64, 4096, 1040), "stream 4x2 w4"), (("nn", 33, 8192, 1152), "stream 4x2 w4"),
    (("tn", 33, 4103, 144), "64x64"), (("tn", 64, 8195, 256), "64x64"), (("nt", 64, 4096, 1024), "64x64"),
    (("tn", 64, 8193, 1040), "64x64"), (("nt", 33, 21504, 2064), "64x128 k2"),
]


@pytest.mark.parametrize("layout,M,N,K", [c for c, _ in CASES])
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

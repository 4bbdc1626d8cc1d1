"""Decoded-operand GEMM in 64- and 128-row tiles: every tile and K-group
configuration at sizes whose last tile, last stage, last slice and last pair
of blocks are partial (K / 16 odd: the last row ends inside a 16-byte chunk),
both scale layouts and output types, against the oracle to the GEMM bar.  The
configurations named per case are checked on the host
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

# (layout, M, N, K), tile and K groups
CASES = [
    (("nt", 71, 272, 16), "64x64"), (("tn", 129, 353, 80), "64x64"),
    (("nt", 68, 352, 1680), "64x64 k2"), (("tn", 68, 353, 1680), "64x64 k2"),
    (("nt", 71, 9392, 16), "64x128"), (("nn", 71, 9392, 272), "64x128"), (("tn", 129, 17889, 528), "64x128"),
    (("nt", 75, 9504, 1264), "64x128 k2"), (("tn", 75, 9506, 1264), "64x128 k2"),
    (("nt", 73, 17888, 48), "128x128"), (("tn", 1100, 4103, 272), "128x128"), (("nn", 1030, 4112, 144), "128x128"),
    (("nt", 777, 4096, 1040), "128x128"), (("tn", 777, 4099, 1040), "128x128"),
    (("nt", 66, 17360, 2512), "128x128 k2"), (("tn", 66, 17366, 2512), "128x128 k2"),
    (("nt", 300, 512, 512), "64x64"), (("nn", 200, 1024, 768), "64x64"),      # K % 256 == 0
]


@pytest.mark.parametrize("layout,M,N,K", [c for c, _ in CASES])
def test_small_tiles(layout, M, N, K):
    say("mid gemm", layout, M, N, K)
    x = synthetic.activation(21, M, K, 0.01, 50.0)
    w = synthetic.weight(22, N, K)
    xq = oq.quantize_1d(x, 1, osc.amax(x))
    X = oq.decoded_1d(xq[0], xq[1], 1)
    if layout != "tn":
        wq = oq.quantize_2d(w, osc.amax(w))
        b, bs, db = wq[0], wq[1], wq[3]
        W = oq.decoded_2d(b, bs)
    else:
        b, bs, db = oq.quantize_1d(w, 1, osc.amax(w))[:3]
        W = oq.decoded_1d(b, bs, 1)
    al = ogemm.alpha(xq[2], db)
    args = (u8_to_dev(xq[0]), u8_to_dev(xq[1]), f32_scalar_dev(xq[2]), u8_to_dev(b), u8_to_dev(bs),
            f32_scalar_dev(db))
    guard = torch.full((M * N + 4096,), 7.25, dtype=torch.float32, device="cuda")
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

"""Probe-matched GEMM: the small and the large tile on the same raw operands
at the edges of the exact paths.  The operands of 64 x 64 outputs repeat over
the large launch, so every output of both has its expected value from the
oracle's model of the 64 x 64 block."""

import numpy as np
import pytest
import torch

import paper_2609_02846_amd as ue
from oracle import quantize as oq
from tests.gpu_util import f32_scalar_dev, host, say, u8_to_dev
from tests.test_gpu_gemm_pm import _ref

pytestmark = pytest.mark.gpu


def _operands(rows, K, tiled, e_top, inner, gap, seed):
    """Blocks 0, 2 of each group at the largest block sum (nibbles 6, scale
    integer 15), block 1 (and 3) of odd products `inner` binades below its
    pair's first block, the second pair `gap` binades below the first; every
    fourth row (second tile) flat."""
    rng = np.random.default_rng(seed)
    nb = K // 16
    odd = rng.choice(np.array([0x1, 0x3, 0x7, 0x9, 0xB, 0xF], np.uint8), (rows, nb, 16))
    nib = np.where((np.arange(nb) % 2 == 1)[None, :, None], odd, np.uint8(7)).reshape(rows, K)
    n = rows // 16 if tiled else rows
    e = np.full((n, nb), e_top, np.int64)
    e[:, 1::4] -= inner
    e[:, 2::4] -= gap
    e[:, 3::4] -= gap + inner
    e[::(2 if tiled else 4), :] = e_top
    return (nib[:, 0::2] | (nib[:, 1::2] << 4)).astype(np.uint8), ((e << 3) | 7).astype(np.uint8)


# K = 144: a partial last group; inner_a + inner_b <= 4 takes the pair path
# whatever the distance between the pairs, 5 the binary64 path; a row of more
# than 16 binades (inner + gap) the integer path
@pytest.mark.parametrize("K,inner_a,inner_b,gap", [(128, 3, 1, 0), (144, 4, 0, 12), (128, 2, 2, 14), (144, 3, 2, 0),
                                                   (128, 0, 4, 16), (144, 4, 0, 13), (128, 2, 0, 20)])
def test_both_tiles_at_the_path_bounds(K, inner_a, inner_b, gap):
    say("gemm_pm tiles", K, inner_a, inner_b, gap)
    pay_a, sa = _operands(64, K, False, 26, inner_a, gap, 31)
    pay_b, sb = _operands(64, K, True, 14, inner_b, 0, 32)
    A, B = oq.decoded_1d(pay_a, sa, 1), oq.decoded_2d(pay_b, sb)
    want = _ref(A, B, np.float32(1.0), 0, [(m, n) for m in range(64) for n in range(64)]).reshape(64, 64)
    one = f32_scalar_dev(1.0)
    for rep in (1, 33):                  # 64 x 64 tiles; 17 x 17 tiles of 128 x 128, the last ones half empty
        a, s, b, t = (u8_to_dev(np.tile(v, (rep, 1))) for v in (pay_a, sa, pay_b, sb))
        c = ue.gemm_pm("nt", 64 * rep, 64 * rep, K, a, s, one, b, t, one, grid=0)
        torch.cuda.synchronize()
        assert np.array_equal(host(c), np.tile(want, (rep, rep))), f"{rep} x {rep} blocks"

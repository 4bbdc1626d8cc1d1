"""Host side of the library calls, without a device: what they launch and in
what order (see host_launches.py)."""

import pytest

from tests import test_gpu_gemm_kernels as kernels
from tests import test_gpu_gemm_mid as small_tiles
from tests import test_gpu_gemm_padded as padded
from tests import test_gpu_gemm_skinny as few_rows
from tests import test_gpu_large as large
from tests.host_launches import amax_call, gemm_call, launches, routes, together

# Calls of several launches that pass data through a library workspace:
# (what, call, launches)
CHAINS = [
    ("split tiles", gemm_call("nt", 4096, 4352, 1024), 2),
    ("split tiles, E8M0", gemm_call("nt", 4096, 4352, 1024, fmt="e8m0", block=32), 2),
    ("codes of blocks of 32", gemm_call("nt", 2048, 2048, 1024, block=32), 2),
    ("codes of blocks of 32, then split tiles", gemm_call("nt", 4096, 4352, 1024, block=32), 3),
    ("codes of blocks of 32, probe-matched", gemm_call("nt", 512, 512, 512, block=32, entry="pm"), 2),
    ("partial maxima", amax_call(1 << 20), 2),
]


@pytest.mark.parametrize("what,call,n", CHAINS, ids=[c[0] for c in CHAINS])
def test_calls_from_several_threads_keep_their_launches_together(what, call, n):
    """Threads that share a stream share its workspaces: a call's launches
    have to be enqueued with no other call's between them, or one would read
    what the other wrote."""
    status, kernels = launches([call])[0]
    assert status == 0 and len(kernels) == n, kernels
    assert together(4, 6, call) == (0, 24, 0)


@pytest.mark.parametrize("N", [(1 << 29) - 48, (1 << 29) - 32, (1 << 29) - 16, 1 << 29, 1 << 31])
@pytest.mark.parametrize("M", [1, 64])
def test_few_rows_of_very_many_columns_launch(M, N):
    """The streaming kernel takes 8 work-items per column, so that from 2^29
    columns on it would not fit a launch dimension; the general kernel does."""
    (status, kernels), = launches([gemm_call("nt", M, N, 16, out="bf16")])
    assert status == 0
    assert [k.split("<")[0] for k, _, _ in kernels] == ["gemm_fp4_skinny_kernel" if N <= (1 << 29) - 32
                                                        else "gemm_fp4_kernel"]


@pytest.mark.parametrize("out", ["f32", "bf16"])
def test_products_of_ragged_k_take_no_workspace(out):
    """A product whose K is not a multiple of 256 runs the same kernels on a
    capturing stream that has no workspace, in an eager call and in the
    allocation-free one, so that their results are equal."""
    for case, names in padded.CASES:
        calls = [gemm_call(*case, out=out, stream=1, capturing=True), gemm_call(*case, out=out, stream=2),
                 gemm_call(*case, out=out, entry="noalloc")]
        assert routes(calls) == [names] * 3, case


def test_few_rows_leave_the_streaming_kernel_only_above_32():
    """More than 32 rows: small tiles once the workgroups of 32 weight rows
    outnumber the 256 CUs or K is at most 1024, unless the weight is too large
    for them (2^31 bytes)."""
    stream = lambda M, N, K: routes([gemm_call("nt", M, N, K)])[0][0].startswith("stream")  # noqa: E731
    for M in (1, 16, 17, 32):
        assert all(stream(M, N, K) for N in (16, 8192, 8208, 65536) for K in (16, 1024, 1040, 8192))
    for M in (33, 64):
        assert all(stream(M, N, K) == (N <= 8192 and K > 1024) for N in (16, 8192, 8208, 65536)
                   for K in (16, 1024, 1040, 8192))
        assert stream(M, 131072, 32768)


def test_gemms_run_on_the_kernels_the_gpu_tests_name():
    """The choice of kernel rests on fitted times: a test that is about one
    kernel has to be at sizes that run on it (256 CUs)."""
    for module in (few_rows, small_tiles):
        for entry in ("gemm", "noalloc"):
            assert routes([gemm_call(*c, entry=entry) for c, _ in module.CASES]) == [[k] for _, k in module.CASES]
    for case, names in kernels.CASES:
        fmt, block = case[4:]
        calls = [gemm_call(*case[:4], out=out, fmt=fmt, block=block) for out in ("f32", "bf16")]
        if fmt == "ue5m3" and block == 16:
            calls.append(gemm_call(*case[:4], entry="noalloc"))
        assert routes(calls) == [names] * len(calls), case
    for case, names in kernels.SMALLEST:
        assert routes([gemm_call(*case), gemm_call(*case, fmt="e4m3")]) == [names] * 2, case
    for case, name in large.OPERAND_CASES:
        assert routes([gemm_call(*case)]) == [[name]], case
    for case, name in large.OUTPUT_CASES:
        assert routes([gemm_call(*case), gemm_call(*case, out="bf16")]) == [[name]] * 2, case

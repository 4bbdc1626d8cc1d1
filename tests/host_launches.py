"""Which kernels a library call launches, found on the host alone: builds
host_launches.cpp (a double of the HIP runtime that records launches; 256
compute units) and feeds it calls."""

import functools
import os
import subprocess
import tempfile

import paper_2609_02846_amd as ue
from paper_2609_02846_amd import build as ue_build

HERE = os.path.dirname(os.path.abspath(__file__))
LAYOUTS = {"nt": 0, "nn": 1, "tn": 2}
KINDS = {"ue5m3": 0, "e4m3": 1, "e8m0": 2}


@functools.lru_cache(maxsize=None)
def _recorder():
    exe = os.path.join(tempfile.mkdtemp(prefix="host_launches_"), "host_launches")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-rdynamic", "-pthread",
                           os.path.join(HERE, "host_launches.cpp"), "-o", exe, "-ldl"])
    if not os.path.exists(ue.LIB_PATH):
        ue_build.build(verbose=False)
    return exe


def _run(lines):
    r = subprocess.run([_recorder(), ue.LIB_PATH], input="\n".join(lines) + "\n", capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stderr
    out = r.stdout.splitlines()
    assert len(out) == len(lines)
    return out


def gemm_call(layout, M, N, K, entry="gemm", out="f32", fmt="ue5m3", block=16, tiled=None, stream=0, capturing=False):
    """Command of one product under the layout's recipe blockings (tiled:
    whether B has tile scales; by default as the layout's recipe)."""
    colT = layout == "tn"
    tiled = (not colT and fmt != "e8m0") if tiled is None else tiled
    a = (1 if colT else 0) + (3 if block == 32 else 0)
    b = (2 if tiled else 1 if layout != "nt" else 0) + (3 if block == 32 else 0)
    if entry == "gemm" and (block == 32 or fmt != "ue5m3"):
        entry = "ex"
    return (f"gemm {entry} {LAYOUTS[layout]} {M} {N} {K} {a} {b} {1 if out == 'bf16' else 0} {KINDS[fmt]} {stream} "
            f"{int(capturing)}")


def amax_call(numel, stream=0, capturing=False):
    return f"amax {numel} {stream} {int(capturing)}"


def launches(calls):
    """Per call: (status, [(kernel with template arguments, grid, block), ...]).
    One process runs all of them in order (workspaces persist)."""
    res = []
    for line in _run(calls):
        status, *rest = line.split(" | ")
        res.append((int(status), [(r.rsplit(" ", 2)[0], *map(int, r.rsplit(" ", 2)[1:])) for r in rest]))
    return res


def together(threads, reps, call):
    """The call from several host threads at once: (status, number of calls,
    how many of them had another call's launch between their own)."""
    w = _run([f"together {threads} {reps} {call}"])[0].split()
    return int(w[0]), int(w[2]), int(w[4])


def short(kernel):
    """A kernel's short name: "large" (256 x 256 tiles; "masked": the
    per-element epilogue, "ragged K": K % 256 != 0), "64x128 k2" (small tiles,
    K groups), "stream 2x1 w8" (few rows: row groups, weight-row groups,
    waves), "staged", "general", "sum" (split tiles), "codes" (blocks of 32),
    "pm 128" (probe-matched tile), "mx"."""
    name, _, rest = kernel.partition("<")
    a = [w.strip() == "true" if w.strip() in ("true", "false") else int(w) for w in rest.rstrip(">").split(",") if w]
    if name == "gemm_fp4_reg_kernel":
        return "large" + ("" if a[2] else " masked") + (" ragged K" if a[3] else "")
    if name == "gemm_fp4_mid_kernel":
        return f"{64 * a[1]}x{64 * a[2]}" + (" k2" if a[3] == 2 else "")
    if name == "gemm_fp4_skinny_kernel":
        return f"stream {a[1]}x{a[2]} w{a[3]}"
    if name == "gemm_pm_kernel":
        return f"pm {64 * a[1]}"
    if name == "gemm_mx_kernel":
        return "mx" + ("" if a[1] else " masked")
    return {"gemm_fp4_dma_kernel": "staged", "gemm_fp4_kernel": "general", "gemm_split_sum_kernel": "sum",
            "copy_scales_kernel": "codes"}.get(name, name)


def routes(calls):
    """The short kernel names of each call, all of which must succeed."""
    res = launches(calls)
    assert all(status == 0 for status, _ in res), res
    return [[short(k) for k, _, _ in kernels] for _, kernels in res]

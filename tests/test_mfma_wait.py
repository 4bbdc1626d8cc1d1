"""The E8M0 GEMM issues its products as instructions the compiler does not
model, so it does not keep accesses to their accumulators clear of products
still in flight; the kernel's own wait states have to.  Checked on the built
library: nothing but products touches an accumulator register within the
product's latency, and the stage loop closes only after it (a move that the
compiler places on the loop's back edge is then safe too)."""

import os
import re
import struct
import subprocess

import pytest

import paper_2609_02846_amd as ue
from paper_2609_02846_amd import build as ue_build

LLVM = "/opt/rocm/llvm/bin"
# A product of 16 passes (FP8 forms; FP4 takes 8) may be followed by a VALU
# access of its result after this many wait states.
WAIT = 20


def _code_objects(path):
    """The gfx950 code objects of the offload bundles in the library."""
    data, magic = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        p = at + len(magic)
        n, = struct.unpack_from("<Q", data, p)
        p += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if name.endswith("gfx950"):
                yield data[at + off:at + off + size]
        at = data.find(magic, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions of every gemm_mx_kernel: (address, text), in order."""
    if not os.path.exists(ue.LIB_PATH):
        ue_build.build(verbose=False)
    tmp, found = tmp_path_factory.mktemp("isa"), {}
    for i, obj in enumerate(_code_objects(ue.LIB_PATH)):
        if b"gemm_mx_kernel" not in obj:
            continue
        f = tmp / f"{i}.o"
        f.write_bytes(obj)
        name = None
        for line in subprocess.run([f"{LLVM}/llvm-objdump", "-d", str(f)], capture_output=True, text=True,
                                   check=True).stdout.splitlines():
            m = re.match(r"[0-9a-f]+ <(.+)>:$", line)
            if m:
                name = m.group(1) if "gemm_mx_kernel" in m.group(1) else None
                if name:
                    found[name] = []
            elif name and "//" in line:
                text, note = line.split("//", 1)
                found[name].append((int(note.split(":")[0], 16), text.strip(), note))
    assert len(found) == 4, found.keys()          # output type x epilogue
    return found


def _states(text):
    m = re.match(r"s_nop (\d+)", text)
    return int(m.group(1)) + 1 if m else 1


def _since_product(code, i):
    """Wait states between the last product before instruction i and i (in
    program order), or None."""
    n = 0
    for _, text, _ in reversed(code[:i]):
        if text.startswith("v_mfma"):
            return n
        n += _states(text)
    return None


def test_accumulators_are_left_alone_while_products_land(kernels):
    for name, code in kernels.items():
        start = code[0][0]
        products = sum(t.startswith("v_mfma_scale") for _, t, _ in code)
        assert products >= 64, name
        loops = 0
        for i, (addr, text, note) in enumerate(code):
            if re.match(r"s_c?branch", text):
                m = re.search(r"\+0x([0-9a-f]+)>", note)
                target = start + (int(m.group(1), 16) if m else 0)
                if target <= addr and any(target <= a < addr and t.startswith("v_mfma") for a, t, _ in code):
                    loops += 1
                    assert _since_product(code, i) >= WAIT, f"{name}: loop closed {_since_product(code, i)} states after"
            elif re.search(r"\ba(\d+|\[)", text) and not text.startswith("v_mfma"):
                n = _since_product(code, i)
                assert n is None or n >= WAIT, f"{name}: {text} {n} wait states after a product"
        assert loops >= 1, name

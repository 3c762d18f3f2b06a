"""The compiler's report on the built kernels: the products that hold 256
accumulators a lane spill no more than a bound.  (Several ways of writing the
accumulators in one instantiation spill them: the float32 dX held stores,
slots and atomics together and took 436 bytes a lane, and 5 to 11% more time.)"""

import os
import re
import struct
import subprocess

import pytest

from paper_2606_18114_amd import ops

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """{demangled kernel: scratch bytes a lane} of the built library."""
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf is needed")
    if not os.path.exists(ops.lib_path()):
        from paper_2606_18114_amd import build
        build.build(verbose=False)
    with open(ops.lib_path(), "rb") as f:
        blob = f.read()
    path = str(tmp_path_factory.mktemp("co") / "kernel.co")
    out = {}
    at = blob.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        (n,) = struct.unpack_from("<Q", blob, pos)
        pos += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, pos)
            target = blob[pos + 24:pos + 24 + idlen].decode()
            pos += 24 + idlen
            if "gfx950" not in target or size == 0:
                continue
            with open(path, "wb") as f:
                f.write(blob[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True,
                                   check=True).stdout
            for m in re.finditer(r"\.private_segment_fixed_size: (\d+).*?\.symbol:\s+(\S+)\.kd",
                                 notes, re.S):
                out[m.group(2)] = int(m.group(1))
        at = blob.find(MAGIC, at + len(MAGIC))
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True,
                           check=True).stdout.split("\n")
    return {n.split("(")[0].replace("void ", ""): b for n, b in zip(names, out.values())}


# (kernel, most scratch bytes a lane).  <g, bfloat16 out, atomics>: the form
# that stores and, where parts have no slots, the one that adds
@pytest.mark.parametrize("kernel,most", [
    *((f"tgemm_bwd_dx_f16_kernel<{g}, {out}, false>", 112)
      for g in (32, 64, 128, 256, 512) for out in ("true", "false")),
    *((f"tgemm_bwd_dx_f16_kernel<{g}, false, true>", 244) for g in (32, 64, 128, 256, 512)),
    ("tgemm_bwd_dw_kernel<false>", 112), ("tgemm_bwd_dw_kernel<true>", 112),
    # <g, code stage, bfloat16 out, shape>: the forward's 256 x 256 and 64 x 128
    # tiles hold everything in registers
    *((f"tgemm_fwd_kernel<{g}, {ss}, {out}, {shape}>", most)
      for g, ss in ((32, 4), (32, 1), (64, 4), (64, 1), (128, 4), (128, 1), (256, 4), (512, 4))
      for out in ("true", "false")
      for shape, most in (("4, 8", 0), ("1, 4", 0), ("2, 4", 32)) if g > 32 or ss == 1 or shape != "2, 4"),
])
def test_scratch(scratch, kernel, most):
    assert scratch["tmk::" + kernel] <= most

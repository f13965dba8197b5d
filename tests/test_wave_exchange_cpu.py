"""Words that the lanes of a wave exchange through LDS without a workgroup
barrier: the order of the accesses has to be given to the compiler.  Checked on
the IR of a kernel that is compiled here (no GPU): every wave barrier stands
between a release and an acquire fence, and the LDS accesses carry one type (a
64-bit view and a 32-bit view of the same words that type-based alias analysis
tells apart could be moved past each other)."""
import os
import re
import subprocess

import pytest

from paper_1808_00128_amd import build


def _device_ir(name, tmp_path):
    out = str(tmp_path / (name + ".ll"))
    cmd = [build.HIPCC, *build.FLAGS, *build.EXTRA_FLAGS.get(name, []), "--cuda-device-only", "-S", "-emit-llvm",
           os.path.join(build.CSRC, name), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(out) as f:
        return f.read()


@pytest.mark.parametrize("name", ["evolve_c16.hip", "inner.hip"])
def test_wave_barriers_stand_between_fences(name, tmp_path):
    lines = [ln.strip() for ln in _device_ir(name, tmp_path).splitlines()]
    at = [i for i, ln in enumerate(lines) if "call void @llvm.amdgcn.wave.barrier()" in ln]
    assert at
    for i in at:
        assert lines[i - 1].startswith('fence syncscope("wavefront") release'), lines[i - 1]
        assert lines[i + 1].startswith('fence syncscope("wavefront") acquire'), lines[i + 1]


def test_column_exchange_has_one_type(tmp_path):
    ir = _device_ir("evolve_c16.hip", tmp_path)
    tags = set(re.findall(r"ptr addrspace\(3\).*?!tbaa !(\d+)", ir))
    names = set()
    for t in tags:
        base = re.search(rf"^!{t} = !{{!(\d+),", ir, re.M).group(1)
        names.add(re.search(rf'^!{base} = !{{!"([^"]+)"', ir, re.M).group(1))
    assert names <= {"omnipotent char"}, names


def test_every_wave_exchange_uses_the_helper():
    for f in sorted(os.listdir(build.CSRC)):
        with open(os.path.join(build.CSRC, f)) as h:
            n = h.read().count("__builtin_amdgcn_wave_barrier")
        assert n == (1 if f == "device_common.hpp" else 0), f

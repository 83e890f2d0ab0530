"""Registers of the built kernels, read from the metadata in libmialign.so: kernels whose speed depends on staying within a
register budget.  A kernel that outgrows it still runs, and every result stays right, so nothing else would show it."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2002_04561_amd as aln

LIB = os.path.join(os.path.dirname(os.path.abspath(aln.__file__)), "libmialign.so")
BIN = "/opt/rocm/llvm/bin/"

pytestmark = pytest.mark.skipif(not os.path.exists(BIN + "llvm-readelf"), reason="no llvm-readelf")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: {key: value}} of every kernel of the library."""
    assert os.path.exists(LIB), "library not built"
    d = tmp_path_factory.mktemp("lib")
    shutil.copy(LIB, d / "lib.so")
    subprocess.run([BIN + "llvm-objdump", "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    found = {}
    for p in sorted(os.listdir(d)):
        if "gfx950" not in p:
            continue
        notes = subprocess.run([BIN + "llvm-readelf", "--notes", p], cwd=d, check=True, capture_output=True, text=True).stdout
        for block in re.split(r"\n  - \.", notes)[1:]:
            keys = dict(re.findall(r"\.?(\w+): +(\S+)", block))
            if "vgpr_count" in keys:
                found[keys["name"]] = keys
    return found


def _named(kernels, pattern):
    got = {n: k for n, k in kernels.items() if re.search(pattern, n)}
    assert got, pattern
    return got


def test_local_lanes_with_codes_do_not_spill(kernels):
    """One pair per lane in 16 bits, local, with codes (mode 1, any gaps, traceback)."""
    for name, k in _named(kernels, r"batch_i16_kernelILi1ELb[01]ELb1E").items():
        assert int(k["vgpr_spill_count"]) == 0, (name, k["vgpr_count"], k["vgpr_spill_count"])


def test_grouped_scores_leave_room_for_five_waves(kernels):
    """The score-only bands in groups that are built for 5 waves a SIMD (last template argument) keep to a fifth of its 512
    registers: else their workgroups are not all resident, whatever the launch holds."""
    got = _named(kernels, r"wf_i32_group_kernelILi\d.*Li4ELb0ELb0ELi5E")
    # 3 modes, linear and affine gaps (float and integer lanes), 5 profiles
    assert len(got) == 45, sorted(got)
    for name, k in got.items():
        assert int(k["vgpr_count"]) <= 96, (name, k["vgpr_count"])

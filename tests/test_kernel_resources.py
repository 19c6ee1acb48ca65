"""Registers of the step kernels, from the metadata that the compiler wrote into the
library built here: none of them may spill vector registers (a spin-orbit instance that
did once gave wrong results) or reserve scratch memory. Exceptions: the persistent batch
kernel in FP64, which holds a whole step, and two forms of the force that reserve (and
don't access) it for scalars which the compiler then keeps in vector lanes."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1801_10233_amd import spinlat as sl

BIN = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> (scratch bytes per lane, spilled vector registers)"""
    if not os.path.exists(sl.LIB_PATH):
        pytest.skip("library not built")
    d = tmp_path_factory.mktemp("kernels")
    lib = shutil.copy(sl.LIB_PATH, d)
    subprocess.run([f"{BIN}/llvm-objdump", "--offloading", os.path.basename(lib)], cwd=d, check=True,
                   capture_output=True)
    out = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        notes = subprocess.run([f"{BIN}/llvm-readelf", "--notes", f], cwd=d, check=True,
                               capture_output=True, text=True).stdout
        for k in notes.split("  - .agpr_count:")[1:]:
            def field(name):
                return re.search(rf"\.{name}:\s+(\S+)", k).group(1)
            out[field("symbol")] = (int(field("private_segment_fixed_size")),
                                    int(field("vgpr_spill_count")))
    names = subprocess.run(["c++filt"], input="\n".join(n.replace(".kd", "") for n in out),
                           check=True, capture_output=True, text=True).stdout.splitlines()
    return dict(zip(names, out.values()))


RESERVED = {"void sl::k_force<float, 6, 1, 12>", "void sl::k_force<float, 7, 1, 12>"}


@pytest.mark.parametrize("family,least", [("k_force<", 300), ("k_pair<", 16), ("k_eam_density<", 2),
                                          ("k_spin_phase<", 200), ("k_spin_tail<", 20), ("k_spin_lds<", 12),
                                          ("k_batch_force<", 50), ("k_batch_spin<", 10),
                                          ("k_batch_tail<", 4)])
def test_step_kernels_use_no_scratch(kernels, family, least):
    mine = {n: v for n, v in kernels.items() if "sl::" + family in n}
    assert len(mine) >= least
    bad = {n.split("(")[0]: v for n, v in mine.items() if v != (0, 0)}
    assert all(v[1] == 0 for v in bad.values()) and set(bad) <= RESERVED, bad

"""CPU checks of the sweep's compiled code, as for the other kernel files."""

import os
import subprocess

import pytest

from tests.test_library_cpu import ROOT, _kernel_argument_records, _misplaced_copies, _record_layouts

SOURCES = ["rips_sweep.hip", "rips_sweep_dim.hip"]
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.parametrize("src", SOURCES)
@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_sweep_argument_layouts_match_between_host_and_device(src):
    host, dev = _record_layouts(src, "host"), _record_layouts(src, "device")
    wanted = _kernel_argument_records(src)
    checked = 0
    for t, lay in host.items():
        if t.replace("struct ", "").replace("rips::", "") in wanted:
            assert dev.get(t) == lay, (t, lay, dev.get(t))
            checked += 1
    assert checked >= 1


@pytest.mark.parametrize("src", SOURCES)
@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_sweep_has_no_register_copy_before_exec_restore(tmp_path, src):
    out = str(tmp_path / "k.s")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I",
                        os.path.join(ROOT, "include"), "--cuda-device-only", "-S", src, "-o", out],
                       capture_output=True, text=True, timeout=600,
                       cwd=os.path.join(ROOT, "paper_1908_02518_amd", "csrc"))
    assert r.returncode == 0, r.stderr[-2000:]
    hits = _misplaced_copies(open(out).read())
    assert not hits, hits[:5]

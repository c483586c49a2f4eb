"""Register budget of the sampling kernels, checked at compile time on the CPU.

A source edit (or the machine scheduler chosen for sample.hip in build_lib) can
make the compiler spill into scratch memory inside a token loop, which slows a
kernel by a large factor, or drains the loads it has requested ahead, while
every parity test still passes.  The tests compile the sources for gfx950 with
the library's own flags.

* The sampler over weight rows, which most sweeps run: every instance keeps the
  wavefronts per SIMD that it is budgeted for, without scratch; with word
  associations the instances of at most four topics per lane may spill 48 bytes
  (a few values per chunk of tokens).
* The samplers over count rows: for every plain instance the sweeps launch with
  16-bit shadow-base rows and without the debug trace, no scratch memory, and at
  most 128 VGPRs (4 wavefronts per SIMD) for up to 8 topics per lane.
"""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_1510_06549_amd import build_lib

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def resource_usage(src):
    """{kernel name: {"VGPRs": n, "ScratchSize": bytes}} from the compiler's
    resource remarks for one source, compiled with its build flags."""
    flags = [f for f in build_lib.source_flags(src) if f not in ("-fPIC", "-Wall")]
    cmd = [HIPCC, *flags, "--cuda-device-only", "-c", os.path.join(build_lib.CSRC, src),
           "-o", os.devnull, "-Rpass-analysis=kernel-resource-usage"]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert out.returncode == 0, out.stderr[-2000:]
    usage, name = {}, None
    for line in out.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            usage[name] = {}
            continue
        m = re.search(r"remark:\s+(VGPRs|ScratchSize \[bytes/lane\]): (\d+)", line)
        if m and name:
            usage[name][m.group(1).split()[0]] = int(m.group(2))
    return usage


@pytest.fixture(scope="module")
def usage_of():
    """resource_usage of every sampler source, compiled side by side."""
    srcs = ["sample.hip", "sample_assoc.hip", "sample_rows.hip", "sample_rows_assoc.hip"]
    with ThreadPoolExecutor(len(srcs)) as pool:
        return dict(zip(srcs, pool.map(resource_usage, srcs)))


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("src", ["sample_rows.hip", "sample_rows_assoc.hip"])
def test_weight_row_sampler_keeps_its_registers(usage_of, src):
    assoc = "assoc" in src
    name = re.compile(r"k_sample_rowsILi(\d+)ELi(\d+)ELb%dE" % assoc)
    seen = {}
    for n, u in usage_of[src].items():
        if m := name.search(n):
            seen[int(m.group(1)), int(m.group(2))] = u
    kpls = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 13, 14, 16}  # topics per lane
    # (64 lanes: only for more than 128 topics)
    assert set(seen) == {(lanes, k) for lanes in (16, 32, 64) for k in kpls
                         if lanes < 64 or k > 2}
    for (lanes, kpl), u in seen.items():
        # 512 VGPRs a lane of a SIMD, shared by 5, 4 or 3 wavefronts in units of 8
        most = 96 if kpl <= 4 else 128 if kpl <= 13 else 168
        assert u["VGPRs"] <= most, (lanes, kpl, u)
        assert u.get("ScratchSize", 0) <= (48 if assoc and kpl <= 4 else 0), (lanes, kpl, u)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_sampler_hot_instances_do_not_spill(usage_of):
    usage = usage_of["sample.hip"]
    # k_sample<KPL, TRACE = false, WIDE = false, BIGQ>
    hot = {n: u for n, u in usage.items() if re.search(r"k_sampleILi\d+ELb0ELb0ELb[01]E", n)}
    assert len(hot) == 12, sorted(usage)  # KPL in {1, 2, 4, 8, 12, 16}, both address widths
    for name, u in hot.items():
        assert u.get("ScratchSize", 0) == 0, (name, u)
        kpl = int(re.search(r"k_sampleILi(\d+)E", name).group(1))
        if kpl <= 8:
            assert u["VGPRs"] <= 128, (name, u)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_association_sampler_benchmark_instance_does_not_spill(usage_of):
    """The word-association sampler over count rows at 8 topics per lane and 4
    sources per word (K = 500 with four sources) runs at 3
    wavefronts per SIMD: no scratch memory and at most 170 VGPRs."""
    usage = usage_of["sample_assoc.hip"]
    hot = {n: u for n, u in usage.items() if re.search(r"k_sample_assocILi8ELi4ELb0ELb[01]E", n)}
    assert len(hot) == 2, sorted(usage)
    for name, u in hot.items():
        assert u.get("ScratchSize", 0) == 0 and u["VGPRs"] <= 170, (name, u)

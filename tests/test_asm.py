"""What the compiler makes of places whose speed or correctness hangs on the order
of memory instructions (gfx950 assembly of single kernels; no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2607_08991_amd import build

SM_GATEUP = [("uint16_t", mt) for mt in (1, 2, 3, 4)] + [("float", mt) for mt in (1, 2, 3, 4)]


@pytest.fixture(scope="module")
def sm_gateup(tmp_path_factory):
    """Memory and barrier instructions of each sm_gateup_kernel, in order."""
    folder = tmp_path_factory.mktemp("asm")
    src, out = str(folder / "k.hip"), str(folder / "k.s")
    with open(src, "w") as f:
        f.write('#include <hip/hip_runtime.h>\n#include "prefill.hpp"\n')
        for t, mt in SM_GATEUP:
            f.write(f"template __global__ void sats::sm_gateup_kernel<{t}, {mt}>(sats::PfArgs, int);\n")
    cmd = [a for a in build.command(out) if a not in build.SOURCES and a not in ("-shared", "-fPIC")]
    subprocess.run(cmd + ["-I", build.CSRC, "--cuda-device-only", "-S", src], check=True, capture_output=True)
    kernels, name = {}, None
    for line in open(out):
        m = re.match(r"_ZN4sats16sm_gateup_kernelI(\w)Li(\d)E\w*:", line)
        if m:
            name = ({"t": "uint16_t", "f": "float"}[m[1]], int(m[2]))
            kernels[name] = []
        elif "s_endpgm" in line:
            name = None
        elif name and re.search(r"\b(buffer_load|s_waitcnt|s_barrier)", line):
            kernels[name].append(line.strip())
    return kernels


@pytest.mark.parametrize("t,mt", SM_GATEUP)
def test_the_route_lookup_delays_no_stage(sm_gateup, t, mt):
    """sm_gateup_kernel reads a row's id first, then issues four of its five stages or
    more (three loads each), and only then waits for the id and reads its table entry,
    in front of the first barrier (whose wait counts that load)."""
    ins = sm_gateup[(t, mt)]
    first_stage = next(i for i, l in enumerate(ins) if l.endswith("lds"))
    assert any("buffer_load_dword " in l for l in ins[:first_stage])
    assert not any("vmcnt" in l for l in ins[:first_stage]), ins[:first_stage]
    entry = next(i for i, l in enumerate(ins) if "buffer_load_ubyte" in l)
    barrier = next(i for i, l in enumerate(ins) if "s_barrier" in l)
    assert entry < barrier
    assert sum(l.endswith("lds") for l in ins[:barrier]) == 15
    issued = sum(l.endswith("lds") for l in ins[:entry])
    waits = [int(m[1]) for l in ins[:entry] for m in [re.search(r"vmcnt\((\d+)\)", l)] if m]
    assert issued >= 12 and waits == [issued], ins[:entry]  # (only the id is waited for)

"""Registers and scratch of the built kernels, from the library's own
metadata: what the rules that choose between kernels take for granted."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
FULL, RWMH, MALA, HMC = 1, 0, 1, 2


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(name, template arguments) -> {"vgpr", "spill"} for every kernel."""
    from paper_2409_07148_amd.restore import LIB_PATH
    blob = open(LIB_PATH, "rb").read()
    out, at = {}, 0
    work = tmp_path_factory.mktemp("objects")
    while (at := blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        n, = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + length].decode()
            p += 24 + length
            if "gfx950" in name and size:
                f = work / f"{at}.co"
                f.write_bytes(blob[at + off:at + off + size])
                text = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
                for part in text.split("  - .agpr_count:")[1:]:
                    def get(key):
                        return re.search(rf"\.{key}:\s+(\S+)", part).group(1)
                    m = re.match(r"_ZN7restore\d+([a-z_]+_kernel)I(.*?)EEv", get("symbol").strip("'"))
                    if m:
                        args = tuple(int(v) for v in re.findall(r"L[ib](\d+)E", m.group(2) + "E"))
                        out[m.group(1), args] = {"vgpr": int(get("vgpr_count")), "spill": int(get("vgpr_spill_count"))}
        at += 24
    return out


def test_one_lane_drain_has_no_other_forms_registers(kernels):
    # the same step as the step kernel's, one lane a chain: about its registers
    for d in range(1, 17):
        for local in (RWMH, MALA, HMC):
            step = kernels["step_kernel", (d, FULL, local, 0, 0, 0, 0)]["vgpr"]
            drain = kernels["drain_kernel", (d, FULL, local, 0, 0, 0)]["vgpr"]
            assert drain <= 1.15 * step + 8, (d, local, drain, step)


def test_kernels_that_ask_for_waves_do_not_spill(kernels):
    # the split kernels are compiled for a number of waves a SIMD
    split = {k: v for k, v in kernels.items() if k[0] == "step_kernel" and k[1][6] == 1}
    assert len(split) == 13 * 3 * 2 + 2 * 2   # d = 4..16, three moves, restore and MH; 8-D learned mu
    batch = {k: v for k, v in kernels.items() if k[0].startswith("batch_") and k[1][-1] == 1}
    assert len(batch) == 20
    assert not {k: v for k, v in {**split, **batch}.items() if v["spill"]}


def test_kernels_over_lanes_do_not_spill(kernels):
    for d in range(1, 17):
        for local in (RWMH, MALA, HMC):
            for kernel, args in (("drain_wide_kernel", ()), ("step_pre_kernel", (4,)), ("drain_pre_kernel", (4,))):
                assert kernels[kernel, (d, FULL, local) + args]["spill"] == 0, (kernel, d, local)

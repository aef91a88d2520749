"""The long-context attention kernel on the host (no GPU): which calls it takes,
and its loads and waits as compiled for gfx950 (the compiler's assembly of this
repository's source)."""
import re
import subprocess

import pytest

from paper_2605_08755_amd import build
from routes import attention_long

LOADS = 8  # load instructions of one step's keys, and of its values


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "decode.s"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-Wall")]
    subprocess.run([build.HIPCC, *flags, "--cuda-device-only", "-S", "-I", build.ROOT + "/include", "-I",
                    build.PKG + "/csrc", "-o", str(out), build.PKG + "/csrc/decode.hip"], check=True,
                   capture_output=True)
    return out.read_text()


@pytest.mark.parametrize("R", [1, 2, 4, 8])
def test_next_step_stays_in_flight(assembly, R):
    """The loop over steps: each request is the keys' loads and then the values',
    as the counted wait for the keys assumes, and no wait of the loop reaches
    into the step that was requested last."""
    body = re.search(r"^_ZN3laq\S*attn_qkv_flash_kernelILi%dE\S*:(.*?)\.amdhsa_kernel" % R, assembly, re.S | re.M)[1]
    loops = [b for b in re.split(r"^\.LBB", body, flags=re.M) if "Loop" in b and "mfma" in b]
    assert len(loops) == 1
    events = []  # K / V: a load of keys / values; an integer: loads that a wait leaves in flight
    for line in loops[0].splitlines():
        if re.match(r"\s+(buffer|global|flat)_load", line):
            events.append("K" if line.rstrip().endswith(" lds") else "V")
        elif m := re.search(r"vmcnt\((\d+)\)", line):
            events.append(int(m[1]))
    loads = [e for e in events if isinstance(e, str)]
    assert loads == 2 * (LOADS * ["K"] + LOADS * ["V"])
    waits = [e for e in events if isinstance(e, int)]
    assert waits.count(3 * LOADS) == 2 and min(waits) >= 2 * LOADS, events


# (query heads, key/value heads, pos) -> kernel: both sides of the measured lines.
@pytest.mark.parametrize("shape,long", [
    ((2, 2, 8191), False), ((2, 2, 8192), True), ((32, 8, 12287), False), ((32, 8, 12288), True),
    ((128, 128, 12288), True), ((129, 129, 12288), False), ((516, 129, 40000), False), ((1032, 129, 12288), True),
    ((149, 149, 12288), False), ((150, 150, 12288), True), ((256, 256, 12288), True), ((300, 300, 12288), False),
    ((383, 383, 12288), False), ((384, 384, 12288), True), ((520, 520, 12288), False), ((2560, 320, 12288), True),
])
def test_long_context_lines(shape, long):
    """More than 128 key/value heads: only where the last round of blocks, one
    to a compute unit, still fills the chip."""
    assert attention_long(*shape) == long

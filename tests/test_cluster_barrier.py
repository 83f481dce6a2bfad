"""The grid barrier of the clustering rounds publishes the stores of every wave
of a block: in the code built for gfx950, each wave waits for its own stores
(vmcnt 0) before the block barrier behind which one lane signals the block's
arrival, and that lane's wave writes L2 back before it signals."""
import os
import re
import subprocess

import pytest

from paper_1410_4803_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def rounds_code(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "cluster.s")
    flags = [f for f in build.HIPCC_FLAGS if f != "-fPIC"]
    subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, "cluster.hip"), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    body = re.search(r"^_ZN2pg11k_cl_rounds\w+:.*?^\.Lfunc_end", text, re.S | re.M).group(0)
    return [l.split(";")[0].strip() for l in body.splitlines()]


def _straight(lines):
    """`lines` up to the first label or branch."""
    for l in lines:
        if l.endswith(":") or l.startswith(("s_branch", "s_cbranch")):
            return
        yield l


def test_arrival_follows_every_waves_stores(rounds_code):
    arrival = next(i for i, l in enumerate(rounds_code) if l.startswith("global_atomic_add"))
    barrier = max(i for i in range(arrival) if rounds_code[i] == "s_barrier")
    before = list(_straight(reversed(rounds_code[:barrier])))
    waits = [i for i, l in enumerate(before) if re.match(r"s_waitcnt.*vmcnt\(0\)", l)]
    stores = [i for i, l in enumerate(before) if re.match(r"(global|flat|buffer)_store", l)]
    assert waits and not (stores and stores[0] < waits[0]), before[:12]
    # the signalling lane: write-back, its end, the arrival
    signal = list(_straight(reversed(rounds_code[:arrival])))
    done = next(i for i, l in enumerate(signal) if re.match(r"s_waitcnt.*vmcnt\(0\)", l))
    assert any(re.match(r"buffer_wbl2.*sc1", l) for l in signal[done:]), signal[:12]

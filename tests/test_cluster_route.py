"""Which form of the clustering a call takes, on the CPU: the library runs in a
child process against stand-ins of the HIP calls that it decides by and
launches through.  Where the cooperative launch of the rounds cannot run or is
turned down, the call merges one pair at a time instead, and no error is left
behind."""
import pytest

import fakehip
from paper_1410_4803_amd import _native

CHILD = r"""
import ctypes, sys
lib = ctypes.CDLL(sys.argv[1])
n = ctypes.c_size_t(0)
m = int(sys.argv[2])
lib.pg_cluster_workspace_bytes(ctypes.c_int64(m), ctypes.byref(n))
p = ctypes.c_void_p(4096)
rc = lib.pg_ibs_cluster(p, p, p, ctypes.c_int64(m), p, p, n, None)
fake = ctypes.CDLL(None)
sys.stdout.flush()
fake.printf(b"rc %d last %d\n", rc, fake.hipGetLastError())
fake.fflush(None)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fakehip.build(tmp_path_factory.mktemp("fake"))


def _calls(fake, case, m=100):
    return fakehip.launches(fake, case, CHILD, _native.LIB_PATH, m)


@pytest.mark.parametrize("m,blocks", [(10, 2), (100, 13), (10000, 256), (24576, 256)])
def test_rounds_run(fake, m, blocks):
    assert _calls(fake, "", m) == ["plain", f"cooperative {blocks}", "plain"]


@pytest.mark.parametrize("m", [2, 9])
def test_few_samples_merge_one_pair_at_a_time(fake, m):
    assert _calls(fake, "", m) == ["plain"] * 3


@pytest.mark.parametrize("case", ["capturing", "occupancy", "masked"])
def test_one_pair_at_a_time(fake, case):
    calls = _calls(fake, case)
    assert calls == ["plain"] * 3           # distances, neighbours, the merge loop


def test_turned_down_launch_merges_one_pair_at_a_time(fake):
    assert _calls(fake, "rejected") == ["plain", "cooperative 13"] + ["plain"] * 3

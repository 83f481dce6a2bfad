"""Which form of the clustering a call takes, on the CPU: the library runs in a
child process against stand-ins of the HIP calls that it decides by and
launches through.  Where the cooperative launch of the rounds cannot run or is
turned down, the call merges one pair at a time instead, and no error is left
behind."""
import os
import subprocess
import sys

import pytest

from paper_1410_4803_amd import _native

FAKE = r"""
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3_t;
static int last, plain;
static int is(const char* what) { const char* s = getenv("CASE"); return s && !strcmp(s, what); }
int hipGetLastError(void) { int e = last; last = 0; return e; }
int hipPeekAtLastError(void) { return last; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipStreamIsCapturing(void* s, int* c) { *c = is("capturing"); return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int t, size_t lds) {
  *n = !is("occupancy"); return 0;
}
int hipExtStreamGetCUMask(void* s, uint32_t words, uint32_t* mask) {
  uint32_t on = is("masked") ? 4 : 8;
  for (uint32_t w = 0; w < words; ++w) mask[w] = w < on ? ~0u : 0u;
  return 0;
}
int hipEventCreateWithFlags(void** e, unsigned f) { *e = (void*)8; return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { return 0; }
int hipEventRecord(void* e, void* s) { return 0; }
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* s) { return 0; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** s) {
  memset(g, 0, sizeof *g); memset(b, 0, sizeof *b); *lds = 0; *s = 0;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** a, size_t lds, void* s) {
  printf("plain\n"); return 0;
}
int hipLaunchCooperativeKernel(const void* f, dim3_t g, dim3_t b, void** a, unsigned lds, void* s) {
  printf("cooperative %u\n", g.x);
  if (is("rejected")) { last = 720; return 720; }
  return 0;
}
"""

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
    d = tmp_path_factory.mktemp("fake")
    (d / "fake.c").write_text(FAKE)
    out = str(d / "libfake.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", str(d / "fake.c"), "-o", out], check=True)
    return out


def _calls(fake, case, m=100):
    env = dict(os.environ, CASE=case)
    env["LD_PRELOAD"] = ":".join(x for x in (fake, env.get("LD_PRELOAD", "")) if x)
    r = subprocess.run([sys.executable, "-c", CHILD, _native.LIB_PATH, str(m)], env=env,
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    lines = r.stdout.split("\n")
    assert "rc 0 last 0" in lines, r.stdout
    return [l for l in lines if l.startswith(("plain", "cooperative"))]


@pytest.mark.parametrize("m,blocks", [(100, 13), (10000, 256)])
def test_rounds_run(fake, m, blocks):
    assert _calls(fake, "", m) == ["plain", f"cooperative {blocks}", "plain"]


@pytest.mark.parametrize("case", ["capturing", "occupancy", "masked"])
def test_one_pair_at_a_time(fake, case):
    calls = _calls(fake, case)
    assert calls == ["plain"] * 3           # distances, neighbours, the merge loop


def test_turned_down_launch_merges_one_pair_at_a_time(fake):
    assert _calls(fake, "rejected") == ["plain", "cooperative 13"] + ["plain"] * 3

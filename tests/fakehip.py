"""Stand-ins of the HIP calls that the library decides by and launches through, for
tests of the host side on the CPU: a child process runs with them preloaded and
prints one line per launch."""
import os
import subprocess
import sys

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



def build(folder) -> str:
    (folder / "fake.c").write_text(FAKE)
    out = str(folder / "libfake.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", str(folder / "fake.c"), "-o", out], check=True)
    return out


def launches(fake: str, case: str, program: str, *args) -> list:
    """The launches of `program`, which ends by printing the call's status and
    HIP's last error (rc, last): both have to be 0."""
    env = dict(os.environ, CASE=case)
    env["LD_PRELOAD"] = ":".join(x for x in (fake, env.get("LD_PRELOAD", "")) if x)
    r = subprocess.run([sys.executable, "-c", program, *map(str, args)], env=env,
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    lines = r.stdout.split("\n")
    assert "rc 0 last 0" in lines, r.stdout
    return [l for l in lines if l.startswith(("plain", "cooperative"))]

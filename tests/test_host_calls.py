"""What the entry points do around their launches, on the CPU: a C program linked
against libgnmr.so with host stand-ins for the HIP runtime (fake_hip.c) that count
launches and fail where told."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2606_00539_amd")

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "gnmr.h"
extern int fake_launches, fake_fail_launches, fake_fail_events;
#define NEED(call) do { gnmr_status r_ = (call); if (r_ != GNMR_OK) { \
  printf("%s: %d %s\n", #call, (int)r_, gnmr_last_error()); exit(2); } } while (0)

/* units of `segs` bf16 segments of `numel` values each */
static gnmr_ctx* context(int units, int segs, int64_t numel) {
  const int64_t S = (int64_t)units * segs;
  gnmr_config cfg = {units, 3, 2, 1, 1e-12, NULL, GNMR_BUDGET_ACTIVE, 0};
  gnmr_segments s = {S, NULL, NULL, NULL, NULL};
  int64_t* off = malloc(sizeof *off * (size_t)(units + 1));
  int64_t* n = malloc(sizeof *n * (size_t)S);
  int32_t* dt = malloc(sizeof *dt * (size_t)S);
  gnmr_ctx* c;
  for (int b = 0; b <= units; ++b) off[b] = (int64_t)b * segs;
  for (int64_t k = 0; k < S; ++k) n[k] = numel, dt[k] = GNMR_BF16;
  s.unit_seg_off = off, s.seg_numel = n, s.seg_dtype = dt;
  NEED(gnmr_init(&c, &cfg, &s, NULL));
  free(off), free(n), free(dt);
  return c;
}

static const void** pointers(int64_t n) {
  const void** p = malloc(sizeof *p * (size_t)n);
  for (int64_t k = 0; k < n; ++k) p[k] = (const void*)(uintptr_t)(4096 + 16 * k);
  return p;
}

static gnmr_status pass(gnmr_ctx* c, int sumsq, const void* const* p) {
  static double out[1 << 16];
  return sumsq ? gnmr_sumsq(c, p, out, NULL) : gnmr_step(c, 1.1, 1.3, p, NULL);
}

static int unbound(int units, int segs, long numel, int sumsq, int prof) {
  gnmr_ctx* c = context(units, segs, numel);
  const void** p = pointers((int64_t)units * segs);
  if (pass(c, sumsq, NULL) != GNMR_E_INVALID) return 10;
  NEED(gnmr_set_profiling(c, prof));
  for (int events = 0; events <= prof; ++events) {
    if (events) fake_fail_events = 1;
    else fake_fail_launches = 1;
    if (pass(c, sumsq, p) != GNMR_E_HIP) return 11;
    fake_launches = 0;
    if (pass(c, sumsq, NULL) != GNMR_E_INVALID || fake_launches) return 12;
  }
  NEED(pass(c, sumsq, p));
  NEED(pass(c, sumsq, NULL));
  NEED(pass(c, !sumsq, NULL));
  fake_fail_launches = 1;  /* the table keeps what it held */
  if (pass(c, sumsq, p) != GNMR_E_HIP || pass(c, sumsq, NULL) != GNMR_OK) return 13;
  free(p);
  return gnmr_destroy(c);
}

static int launches(int units, int segs, long numel, int prof) {
  gnmr_ctx* c = context(units, segs, numel);
  const void** p = pointers((int64_t)units * segs);
  int32_t said = -1;
  NEED(gnmr_set_profiling(c, prof));
  NEED(gnmr_info(c, NULL, NULL, NULL, &said));
  fake_launches = 0;
  NEED(gnmr_step(c, 1.1, 1.3, p, NULL));
  printf("%d %d\n", (int)said, fake_launches);
  free(p);
  return gnmr_destroy(c);
}

int main(int argc, char** argv) {
  long v[5] = {0};
  for (int k = 2; k < argc && k < 7; ++k) v[k - 2] = atol(argv[k]);
  if (!strcmp(argv[1], "unbound")) return unbound((int)v[0], (int)v[1], v[2], (int)v[3], (int)v[4]);
  if (!strcmp(argv[1], "launches")) return launches((int)v[0], (int)v[1], v[2], (int)v[3]);
  return 3;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cc = shutil.which("gcc")
    if cc is None or not os.path.exists(os.path.join(PKG, "libgnmr.so")):
        pytest.skip("gcc or libgnmr.so is missing")
    d = tmp_path_factory.mktemp("host")
    (d / "calls.c").write_text(PROGRAM)
    subprocess.run([cc, "-std=c99", "-Wall", "-Wextra", "-Werror", "-rdynamic", "-I",
                    os.path.join(ROOT, "include"), str(d / "calls.c"),
                    os.path.join(ROOT, "tests", "fake_hip.c"), "-o", str(d / "calls"), "-L", PKG,
                    "-lgnmr", f"-Wl,-rpath,{PKG}"], check=True)

    def run(*args):
        r = subprocess.run([str(d / "calls"), *map(str, args)], capture_output=True, text=True,
                           timeout=60)
        assert r.returncode == 0, (args, r.returncode, r.stdout)
        return r.stdout
    return run


# Pointers that go with the launch (up to 448): in one launch, in launches of their
# own (more than 256 units, or profiling), and of the gradient pass alone.
@pytest.mark.parametrize("units,segs", [(3, 2), (256, 1), (300, 1), (1, 448)])
@pytest.mark.parametrize("sumsq,prof", [(0, 0), (0, 1), (1, 0)])
def test_a_failed_launch_binds_no_pointers(program, units, segs, sumsq, prof):
    """The launch itself leaves the pointers in the device table: after one that
    failed, a step without pointers is refused, and none reads the empty table."""
    program("unbound", units, segs, 5000, sumsq, prof)


# Up to 256 units of up to 6,144 work items of 32,768 values: one launch, or, while
# profiling, K1 and K2 + K3 as one or two.  A step without items has no K1.
@pytest.mark.parametrize("units,numel,plain,profiling", [
    (28, 65536, 1, 2), (256, 24 * 32768, 1, 2), (256, 24 * 32768 + 1, 2, 2), (1, 6144 * 32768, 1, 2),
    (1, 6145 * 32768, 2, 2), (84, 73 * 32768, 1, 3), (257, 10, 2, 2), (1024, 10, 2, 2),
    (1025, 10, 3, 3), (5, 0, 1, 1), (2000, 0, 2, 2)])
def test_info_gives_the_launches_of_a_step(program, units, numel, plain, profiling):
    for prof, want in ((0, plain), (1, profiling)):
        assert program("launches", units, 1, numel, prof).split() == [str(want)] * 2

"""Launch geometry at the largest numbers of heads that validation admits: no launch of any entry point may exceed what the device takes
(rocminfo: a grid of 2^31 - 1 x 65535 x 65535 blocks, 1024 work-items to a block).

The library is loaded in a child process behind a stand-in for the runtime's launch functions that records every launch and starts
nothing, so that the entry points walk their whole launch sequence without a GPU and without memory."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <stddef.h>
#include <stdint.h>
struct dim3 { uint32_t x, y, z; };
static dim3 g_grid, g_block;
static size_t g_shared;
static void *g_stream;
static uint32_t g_log[4096][4];
static int g_n;
extern "C" {
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void *stream) {
  g_grid = grid; g_block = block; g_shared = shared; g_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, void **stream) {
  *grid = g_grid; *block = g_block; *shared = g_shared; *stream = g_stream;
  return 0;
}
int hipLaunchKernel(const void *, dim3 grid, dim3 block, void **, size_t, void *) {
  const uint32_t launch[4] = {grid.x, grid.y, grid.z, block.x * block.y * block.z};
  for (int i = 0; i < 4 && g_n < 4096; ++i) g_log[g_n][i] = launch[i];
  if (g_n < 4096) ++g_n;
  return 0;
}
int hipGetLastError(void) { return 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { return 0; }
int recorded(uint32_t (**log)[4]) { *log = g_log; const int n = g_n; g_n = 0; return n; }
}
"""

CHILD = r"""
import ctypes, sys
stand_in = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)       # ahead of the runtime that torch loads
from paper_2509_24899_amd import hybrid_attn as ha
lib, FAKE = ha._lib(), 0x7F0000001000
ref = ctypes.byref

def problem(B, H, N, d, f32, R):
    return ha.ha_problem(B, H, N, d, ha.HA_F32 if f32 else ha.HA_BF16, 64, R, 0.1, H * N * d, N * d, d, 0, 0, 0, 0)

def check(what, status):
    assert status == ha.HA_OK, (what, status)
    log = ctypes.POINTER(ctypes.c_uint32 * 4)()
    n = stand_in.recorded(ref(log))
    assert n > 0, what
    for i in range(n):
        x, y, z, block = log[i]
        ok = 0 < x < 2 ** 31 and 0 < y <= 65535 and 0 < z <= 65535 and 0 < block <= 1024
        if not ok:
            bad.append((what, f"launch {i} of {n}", (x, y, z), block))

bad = []
for B, H in ((1, 65535), (1, 40000), (1, 21846), (4, 16383), (65535, 1)):
    for d, hid, mid in ((64, 64, 0), (128, 128, 0), (128, 256, 0), (128, 384, 0), (128, 256, 256)):
        for f32 in (False, True):
            for R in (0, 1, 2):
                N = 70
                p, fm = problem(B, H, N, d, f32, R), ha.ha_feature_map(FAKE, None, FAKE, None, hid, hid, 2, 0, FAKE if mid else None, None, mid, 0)
                what = (B, H, d, hid, mid, "f32" if f32 else "bf16", R)
                big = ctypes.c_size_t(1 << 60)
                check(("forward",) + what, lib.hybrid_attn_forward(ref(p), FAKE, FAKE, FAKE, ref(fm), ref(fm), FAKE, FAKE + 0xF00, big, None))
                check(("loss",) + what, lib.hybrid_attn_value_distill_loss(ref(p), FAKE, FAKE, FAKE, ref(fm), ref(fm), 0, FAKE, 2 * FAKE, FAKE,
                                                                          FAKE + 0xF00, big, None))
                g = ha.ha_feature_map_grad(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE)
                check(("gradient",) + what, lib.hybrid_attn_value_distill_grad(ref(p), FAKE, FAKE, FAKE, ref(fm), ref(fm), 0, 0, FAKE, 2 * FAKE, FAKE, FAKE,
                                                                              ref(g), ref(g), FAKE + 0xF00, big, None))
                if R != 1:
                    check(("state",) + what, lib.hybrid_attn_linear_state(ref(p), FAKE, FAKE, ref(fm), FAKE, FAKE, FAKE + 0xF00, big, None))
seen = set()
for b in bad:
    key = (b[0][0],) + b[0][3:] + (b[1],)
    if key not in seen:
        seen.add(key)
        print(*b, flush=True)
sys.exit(1 if bad else 0)
"""


def test_no_launch_exceeds_the_device(tmp_path):
    source, so, child = tmp_path / "stand_in.cpp", tmp_path / "stand_in.so", tmp_path / "child.py"
    source.write_text(STAND_IN)
    child.write_text(textwrap.dedent(CHILD))
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", str(source), "-o", str(so)], check=True)
    run = subprocess.run([sys.executable, str(child), str(so)], cwd=ROOT, env={**os.environ, "PYTHONPATH": ROOT}, capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, (run.stdout + run.stderr)[-6000:]

"""The device queue of tiles (fr_queue.hpp) compiled for the host over a small
shim of the HIP names it uses: a workgroup that finds the queue empty waits as
long as another one works, however much time passes on the clock meanwhile
(the whole hardware queue may be switched out), and gives up after a bounded
number of its own looks when nothing moves."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_12800_amd", "csrc")

SHIM = r"""
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#define __host__
#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
typedef int hipError_t;
typedef void* hipStream_t;
void looked();                  // one look at the queue (the wait between two)
long long wall_clock64();
#define __builtin_amdgcn_s_sleep(n) looked()
template <typename T> T __hip_atomic_load(T* p, int, int) { return *p; }
template <typename T> void __hip_atomic_store(T* p, T v, int, int) { *p = v; }
template <typename T> T atomicAdd(T* p, T v) { T o = *p; *p = o + v; return o; }
template <typename T> T atomicExch(T* p, T v) { T o = *p; *p = v; return o; }
template <typename T, typename U, typename V> T atomicCAS(T* p, U c, V v) { T o = *p; if (o == (T)c) *p = (T)v; return o; }
"""

MAIN = r"""
#include "fr_queue.hpp"
#include <stdio.h>
#include <string.h>
static fr::TileCtl ctl;
static uint32_t state[2];
static uint64_t ring[4];
static int32_t status;
static long long looks, work_looks, now;
static long long slow;  // ticks of the clock per look
void looked() {
  now += slow;
  if (++looks == work_looks) ctl.left = 0;  // the other workgroup ends its tile, the last one
}
long long wall_clock64() { return now; }
int main(int argc, char** argv) {
  (void)argc;
  slow = atoll(argv[1]);
  work_looks = atoll(argv[2]);
  fr::TileQueue Q;
  memset(&Q, 0, sizeof Q);
  Q.state = state;
  Q.ring = ring;
  Q.ctl = &ctl;
  Q.status = &status;
  Q.stuck = FR_ERR_NOTDAG;
  Q.cap = 4;
  fr::open_queue(Q, 2);
  ctl.head = 2;  // both tiles taken, one done, one in another workgroup's hands
  ctl.left = 1;
  state[0] = fr::ST_DONE;
  state[1] = fr::ST_RUNNING;
  const int32_t t = fr::take_tile(Q);
  printf("%d %d %lld\n", t, status, looks);
  return 0;
}
"""


@pytest.fixture(scope="module")
def queue(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("queue")
    os.makedirs(d / "hip")
    (d / "hip" / "hip_runtime.h").write_text(SHIM)
    (d / "hip" / "hip_runtime_api.h").write_text("#include \"hip_runtime.h\"\n")
    (d / "main.cpp").write_text("#include <stdlib.h>\n" + MAIN)
    exe = str(d / "queue")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wno-attributes", f"-I{d}", f"-I{CSRC}", f"-I{os.path.join(ROOT, 'include')}",
                    "-o", exe, str(d / "main.cpp")], check=True)

    def run(slow, work_looks):
        out = subprocess.run([exe, str(slow), str(work_looks)], check=True, capture_output=True, text=True, timeout=120)
        return [int(x) for x in out.stdout.split()]

    return run


@pytest.mark.parametrize("work_looks", [1, 100, 20000])
@pytest.mark.parametrize("slow", [1, 100, 10**9])
def test_waits_for_a_running_tile(queue, slow, work_looks):
    """`slow`: ticks of the 100 MHz clock per look, up to ten seconds."""
    tile, status, looks = queue(slow, work_looks)
    assert (tile, status) == (-1, 0)
    assert looks <= work_looks + 4


def test_gives_up_when_nothing_moves(queue):
    tile, status, looks = queue(1, -1)
    assert tile == -1 and status == -6  # FR_ERR_NOTDAG
    assert looks <= 1 << 20

"""The sharing of a round's candidate slots among a wave's 64 cells
(csrc/slots.h), run on the host: 64 threads in step, the wave's exchanges
emulated.  Whatever the candidate counts, up to 2^31 - 1 a cell, no cell gets
more than it has, together they get no more than the slots, their slots lie one
after another in the cells' order, and where anything is left something is
taken."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_08195_amd", "csrc")
MAX = 2 ** 31 - 1

HARNESS = r"""
#include <pthread.h>
#include <cstdint>
#include <thread>
#include <vector>
#define __device__
#define __forceinline__ inline
static pthread_barrier_t bar;
static int vals[64];
static thread_local struct { unsigned x; } threadIdx;
static int exchange(int v, int from) {
    vals[threadIdx.x] = v;
    pthread_barrier_wait(&bar);
    const int r = vals[from];
    pthread_barrier_wait(&bar);
    return r;
}
static int __shfl(int v, int lane, int) { return exchange(v, lane); }
static int __shfl_up(int v, int o, int) {
    const int l = (int)threadIdx.x;
    return exchange(v, l >= o ? l - o : l);
}
static uint64_t __ballot(bool p) {
    uint64_t m = 0;
    vals[threadIdx.x] = p;
    pthread_barrier_wait(&bar);
    for (int l = 0; l < 64; ++l) m |= (uint64_t)vals[l] << l;
    pthread_barrier_wait(&bar);
    return m;
}
static int __popcll(uint64_t m) { return __builtin_popcountll(m); }
#include "slots.h"
// out: m, base, total of each lane
extern "C" void share(const int* left, int* out) {
    pthread_barrier_init(&bar, nullptr, 64);
    std::vector<std::thread> t;
    for (int l = 0; l < 64; ++l)
        t.emplace_back([=] {
            threadIdx.x = l;
            out[l] = dsmcx::share_slots<256>(left[l], out + 64 + l, out + 128 + l);
        });
    for (auto& x : t) x.join();
    pthread_barrier_destroy(&bar);
}
"""


@pytest.fixture(scope="module")
def share(tmp_path_factory):
    import ctypes
    d = tmp_path_factory.mktemp("slots")
    (d / "h.cpp").write_text(HARNESS)
    # (-fwrapv: signed sums wrap as the GPU's do)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fwrapv", "-Wno-unknown-pragmas", "-shared", "-fPIC", "-pthread", "-I",
                    CSRC, str(d / "h.cpp"), "-o", str(d / "h.so")], check=True)
    lib = ctypes.CDLL(str(d / "h.so"))

    def run(left):
        left = np.ascontiguousarray(left, dtype=np.int32)
        out = np.zeros((3, 64), dtype=np.int32)
        lib.share(ctypes.c_void_p(left.ctypes.data), ctypes.c_void_p(out.ctypes.data))
        return out

    return run


def _counts():
    rng = np.random.default_rng(1)
    yield "none", np.zeros(64)
    yield "full", np.full(64, 4)
    yield "one over", np.r_[5, np.full(63, 4)]
    yield "one cell", np.r_[np.zeros(40), 1000, np.zeros(23)]
    yield "one at the limit", np.r_[np.zeros(63), MAX]
    yield "two to 2^31", np.r_[2 ** 30, 2 ** 30, np.zeros(62)]
    yield "sum wraps to a small number", np.r_[MAX, MAX, 5, np.zeros(61)]
    yield "all at the limit", np.full(64, MAX)
    yield "33 million and more", np.full(64, 2 ** 25 + 1)
    for k in range(4):
        yield f"random {k}", rng.integers(0, [9, 40, 10 ** 6, MAX][k], 64)


@pytest.mark.parametrize("name,left", list(_counts()), ids=lambda x: x if isinstance(x, str) else "")
def test_shares(share, name, left):
    left = left.astype(np.int64)
    m, base, total = (x.astype(np.int64) for x in share(left))
    assert np.all(m >= 0) and np.all(m <= left)
    assert m.sum() <= 256 and np.all(total == m.sum())
    assert np.array_equal(base, np.cumsum(m) - m)
    if left.sum() <= 256:
        assert np.array_equal(m, left)
    else:
        assert np.array_equal(m, np.minimum(left, 256 // np.count_nonzero(left)))

"""CPU checks of launch sizes and buffer sizes (csrc/sidm_plan.hpp, compiled for
the host with g++): kernels with a workgroup per halo are cut into launches
that a grid can hold and that cover every halo once; the room for candidates of
the scattering decisions grows with the room for events; the workgroups of a
tidal-radius pass are shared out by the halos' sizes."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
_SRC = r'''
#include "sidm_plan.hpp"
extern "C" int chunks(long long total, int threads, long long* first, long long* count, int cap) {
    int k = 0;
    sidm::launch_chunks(total, threads, [&](int64_t f, int64_t c) {
        if (k < cap) { first[k] = f; count[k] = c; }
        ++k;
    });
    return k;
}
extern "C" long long room(long long events, long long n, long long free_bytes) {
    return sidm::candidate_room(events, n, free_bytes);
}
extern "C" int tidal_wg(long long n, long long total) { return sidm::tidal_workgroups(n, total); }
extern "C" int cand_bytes() { return (int)sizeof(sidm::CandRec); }
extern "C" long long events0(long long n) { return sidm::default_events(n); }
'''


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    d = tmp_path_factory.mktemp("sidm_launch")
    src, so = str(d / "p.cpp"), str(d / "p.so")
    with open(src, "w") as f:
        f.write(_SRC)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2506_06269_amd", "csrc"), src, "-o", so,
                    "-L", os.path.join(ROCM, "lib"), "-lamdhip64"], check=True)
    return C.CDLL(so)


@pytest.mark.parametrize("threads", [64, 256, 512, 1024])
@pytest.mark.parametrize("total", [1, 4096, (1 << 22) - 1, 1 << 22, 10_000_001, 256 * 33001])
def test_launches_fit_a_grid(L, total, threads):
    first, count = (C.c_longlong * 64)(), (C.c_longlong * 64)()
    L.chunks.argtypes = [C.c_longlong, C.c_int, C.c_void_p, C.c_void_p, C.c_int]
    k = L.chunks(total, threads, first, count, 64)
    assert 1 <= k <= 64
    at = 0
    for q in range(k):
        assert first[q] == at and 0 < count[q] and count[q] * threads < 1 << 32
        at += count[q]
    assert at == total
    assert k == 1 or total * threads > 1 << 31


@pytest.mark.parametrize("n", [2, 1000, 32768, 65536, 1 << 20, 1 << 24])
def test_candidate_room(L, n):
    L.room.restype = L.events0.restype = C.c_longlong
    L.room.argtypes = [C.c_longlong, C.c_longlong, C.c_longlong]
    L.events0.argtypes = [C.c_longlong]
    e0 = L.events0(n)
    assert e0 == max(4096, n // 8)
    events = sorted({1, 4, e0 // 2, e0 - 1, e0, e0 + 1, 2 * e0, 4 * n, 8 * n + 1})
    room = [L.room(e, n, 1 << 50) for e in events]
    assert all(a <= b for a, b in zip(room, room[1:]))
    for e, r in zip(events, room):
        assert r == 4 * e if e < e0 else r == max(4 * e, 2 * n)


def test_candidate_room_where_memory_is_short(L):
    """Two candidates per particle only where what they add to four per event
    slot is at most an eighth of the free memory."""
    L.room.restype = L.events0.restype = C.c_longlong
    L.room.argtypes = [C.c_longlong, C.c_longlong, C.c_longlong]
    L.events0.argtypes = [C.c_longlong]
    n = 1 << 28
    e0 = L.events0(n)
    more = (2 * n - 4 * e0) * L.cand_bytes()
    assert L.room(e0, n, 8 * more) == 2 * n
    assert L.room(e0, n, 8 * more - 8) == 4 * e0
    assert L.room(e0, n, 0) == 4 * e0
    assert L.room(8 * n, n, 0) == 32 * n


@pytest.mark.parametrize("sizes", [[2], [255], [257], [65536], [1 << 24], [50000] * 40, [300] * 7,
                                   [1 << 24] * 3, [100000] + [300] * 500, [1 << 12, 1 << 17] * 32])
def test_tidal_workgroups(L, sizes):
    L.tidal_wg.argtypes = [C.c_longlong, C.c_longlong]
    wg = [L.tidal_wg(n, sum(sizes)) for n in sizes]
    assert all(1 <= w <= -(-n // 256) for w, n in zip(wg, sizes))
    assert sum(w for w in wg if w > 1) <= 256
    if len(sizes) == 1:
        assert wg[0] == min(256, -(-sizes[0] // 256))

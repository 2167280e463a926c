"""Launch shapes of the library's host code at sizes that no test can run: the built objects
are linked with a recording HIP runtime (tests/native/recording_hip.cpp) that refuses a launch
as the real one does, 2^32 work-items or more along x among the reasons, and runs nothing."""
import ctypes
import os
import subprocess

import pytest

from paper_1805_04463_amd import build as hip_build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    objects = [os.path.join(hip_build.BUILD, os.path.splitext(s)[0] + ".o") for s in hip_build.SOURCES]
    if not all(os.path.exists(o) for o in objects):
        hip_build.build()
    path = str(tmp_path_factory.mktemp("rec") / "librecorded.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic",
                    os.path.join(HERE, "native", "recording_hip.cpp"), *objects, "-o", path], check=True)
    L = ctypes.CDLL(path)
    i64, p, sz = ctypes.c_int64, ctypes.c_void_p, ctypes.c_size_t
    L.rec_kernel.restype = ctypes.c_char_p
    L.rec_reply.argtypes = [p, sz]
    L.cs_sprinkle.argtypes = [ctypes.c_int, ctypes.c_double, ctypes.c_uint64, i64, p, p, sz, p]
    L.cs_dalembertian.argtypes = [p, i64, i64, ctypes.c_int, ctypes.c_double, ctypes.c_int, p, p, p, sz, p]
    L.cs_dalembertian_workspace_bytes.argtypes = [i64, ctypes.c_int]
    L.cs_dalembertian_workspace_bytes.restype = sz
    L.cs_longest_chain.argtypes = [p, i64, i64, p, p, i64, p, p, p, sz, p]
    return L


def launches(L, part):
    """(grid x, grid y, block x) of the recorded launches of kernels named *part*."""
    out = []
    for i in range(L.rec_count()):
        if part in L.rec_kernel(i).decode():
            d = (ctypes.c_uint32 * 6)()
            L.rec_dims(i, d)
            assert (d[2], d[4], d[5]) == (1, 1, 1)
            out.append((d[0], d[1], d[3]))
    return out


ANY = 256          # a device pointer; nothing is read
ROOM = 1 << 60     # workspace bytes


@pytest.mark.parametrize("n,count,active", [
    (131072, 1, 2048), (131072, 2, 4096), (131072, 3, 2049), (131072, 8192, 2**24 - 1), (131072, 8192, 2**24),
    (32768, 32768, 2**24), (20000, 65535, 313 * 65535)])
def test_chain_rounds_over_many_words(rec, n, count, active):
    """A launch per round over `active` words: at least a workgroup for each, less than one
    grid row too many."""
    rec.rec_reset()
    survey = (ctypes.c_uint64 * 4)(64 * active, n, active, 0)
    ended = (ctypes.c_uint64 * 8)(64 * active, n, active, 0, 0, 0, 0, 0)
    if (n + 63) // 64 * count > 4096:  # else the first batch covers every word, unseen
        rec.rec_reply(survey, 32)
    rec.rec_reply(ended, 64)
    ends = (ctypes.c_int64 * (2 * count))(*([-1] * count + [n] * count))
    at = ctypes.addressof(ends)
    rc = rec.cs_longest_chain(ANY, n, n, at, at + 8 * count, count, ANY, ANY, ANY, ROOM, None)
    assert rc == 0
    rounds = launches(rec, "k_chain_round")
    assert len(rounds) == 8
    for x, y, threads in rounds:
        assert x * threads < 2**32 and y <= 65535
        assert 0 <= x * y - active < x
        assert y == 1 or active * threads >= 2**31  # one row wherever it does


@pytest.mark.parametrize("n", [8193, 131072, 2**27, 2**27 + 1, 2**29 - 64, 2**29, 2**29 + 1, 2**31 - 1])
@pytest.mark.parametrize("region", range(5))
def test_bucket_placement_of_many_points(rec, region, n):
    """A workgroup for each 64 points.  (The candidates of the 3+1 and 2+1 diamonds, about eight and
    four per point, are a work-item each: their own launch is refused above these sizes, as it
    always was.)"""
    if n > {1: 2**29 + 1, 4: 2**30}.get(region, n):
        return
    rec.rec_reset()
    assert rec.cs_sprinkle(region, 1.2, 7, n, ANY, ANY, ROOM, None) == 0
    (x, y, threads), = launches(rec, "k_bucket_place")
    buckets = (n + 63) // 64
    assert x * threads < 2**32 and y <= 65535
    assert 0 <= x * y - buckets < x
    assert y == 1 or buckets * threads >= 2**30


@pytest.mark.parametrize("counter,last", [(1, 15000), (2, 32768)], ids=["mfma", "mfma_fp4"])
@pytest.mark.parametrize("n", [700, 4096, 4097, 10007, 15000, 15001, 32768, 32769])
def test_dalembertian_tiles_follow_the_workspace(rec, n, counter, last):
    """128-row tiles need room for their second sums above 4096 points: with the 256 bytes that
    are always enough, larger sets keep the 256-row tiles, whose rounding error is smaller than
    that of 128-row tiles with one sum per element."""
    full = rec.cs_dalembertian_workspace_bytes(n, counter)
    assert full == 256 + (8 * n if n <= last else 0)
    for room in (256, full - 1, full):
        if room < 256:
            continue
        rec.rec_reset()
        assert rec.cs_dalembertian(ANY, n, 1 << 10, 4, 1.0, counter, ANY, ANY, ANY, room, None) == 0
        small = n <= 4096 or (n <= last and room == full)
        tiles = -(-n // (128 if small else 256))
        tiles = tiles * (tiles + 1) // 2
        assert len(launches(rec, "k_count_mfmaILi2E" if small else "k_count_mfmaILi4E")) == 1
        (x, y, threads), = launches(rec, "k_count_mfma")
        assert (x, y, threads) == (tiles if small else min(tiles, 256), 1, 256)


@pytest.mark.parametrize("count", [1, 256, 257, 40000, 65535])
def test_chain_survey_workgroups(rec, count):
    """Each workgroup of a survey adds to the same line: at most 256 of them."""
    rec.rec_reset()
    n, words = 65, 2 * count
    survey = (ctypes.c_uint64 * 4)(words, 2, words, 0)
    ended = (ctypes.c_uint64 * 8)(words, 2, words, 0, 0, 0, 0, 0)
    if words > 4096:
        rec.rec_reply(survey, 32)
    rec.rec_reply(ended, 64)
    ends = (ctypes.c_int64 * (2 * count))(*([-1] * count + [n] * count))
    at = ctypes.addressof(ends)
    assert rec.cs_longest_chain(ANY, n, 8, at, at + 8 * count, count, ANY, ANY, ANY, ROOM, None) == 0
    surveys = launches(rec, "k_chain_survey")
    assert len(surveys) == 2
    assert all(x <= 256 and y == 1 and threads == 1024 for x, y, threads in surveys)


@pytest.mark.parametrize("sizes,small,large", [
    ([30] * 60000, 60000, 0), ([512] * 512, 512, 0), ([512] * 511, 0, 511), ([192, 2, 64], 3, 0),
    ([193, 2, 64], 0, 3), ([8192] + [100] * 512, 512, 1), ([8192] + [100] * 511, 0, 512),
    ([513] * 600, 0, 600)])
def test_ensemble_forms(rec, sizes, small, large):
    """Small diamonds leave the kernels that are sized for 8192 points, where they are many or
    alone."""
    rec.rec_reset()
    i64, p, sz = ctypes.c_int64, ctypes.c_void_p, ctypes.c_size_t
    rec.cs_batch_plan.argtypes = [i64, p, ctypes.c_int, ctypes.c_int, p, p, p]
    rec.cs_batch_run.argtypes = [p, p, p, p, p, sz, p]
    n, plan = (ctypes.c_int64 * len(sizes))(*sizes), p()
    assert rec.cs_batch_plan(len(sizes), n, 2, 0, None, None, ctypes.byref(plan)) == 0
    assert rec.cs_batch_run(plan, ANY, ANY, ANY, ANY, ROOM, None) == 0
    for cap, count in ((512, small), (8192, large)):
        for kernel in ("k_sprinkle_mink2_batch", "k_rank_tables", "k_build_batch", "k_count_ranks"):
            seen = launches(rec, f"{kernel}ILi{cap}")
            assert len(seen) == (1 if count else 0), (kernel, cap)
            if count and kernel == "k_sprinkle_mink2_batch":
                assert seen[0] == (count, 1, 128 if cap == 512 else 1024)
    rec.cs_batch_free.argtypes = [p]
    assert rec.cs_batch_free(plan) == 0

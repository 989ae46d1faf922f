"""The samples that split the key sort into buckets.

A bucket of more than 8192 keys is sorted by one workgroup in global memory, in
milliseconds, so the samples have to represent the keys in whatever order the
caller holds the particles: lattices in row order, particles in pairs, sorted ones.
The places come from the library's own header, compiled for the host; the split is
then done here on the keys. On the GPU, keys placed to defeat the samples send most
of them to one bucket, which has to come out in stable order all the same.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CAP, OVER = 8192, 8

PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "sample_sort.hpp"
int main(int argc, char** argv) {
    using namespace pbh;
    const int64_t n = std::atoll(argv[1]), m = (int64_t)ss_buckets(n) * kSsOver;
    std::printf("%d %d\\n", kSsCap, kSsOver);
    for (int64_t j = 0; j < m; ++j) std::printf("%lld\\n", (long long)ss_sample_at(j, n, m));
    return 0;
}
"""


@pytest.fixture(scope="module")
def places(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if cxx is None or not os.path.isdir(os.path.join(rocm, "include", "hip")):
        pytest.skip("no host compiler or HIP headers")
    d = tmp_path_factory.mktemp("places")
    (d / "places.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I",
                    os.path.join(ROOT, "paper_2110_11658_amd", "csrc"), str(d / "places.cpp"), "-o",
                    str(d / "places")], check=True)

    def at(n):
        v = np.array(subprocess.run([str(d / "places"), str(n)], capture_output=True, text=True,
                                    check=True).stdout.split(), dtype=np.int64)
        assert tuple(v[:2]) == (CAP, OVER)
        v = v[2:]
        assert np.all(np.diff(v) > 0) and v[0] >= 0 and v[-1] < n
        return v
    return at


def _spread(v):
    v = v.astype(np.uint64)
    for s, m in ((32, 0x1f00000000ffff), (16, 0x1f0000ff0000ff), (8, 0x100f00f00f00f00f),
                 (4, 0x10c30c30c30c30c3), (2, 0x1249249249249249)):
        v = (v | (v << np.uint64(s))) & np.uint64(m)
    return v


def _keys(pos):
    lo = pos.min(0)
    q = np.minimum(np.floor((pos - lo) * (2.0**21 / (pos - lo).max())), 2**21 - 1).astype(np.int64)
    x, y, z = (_spread(q[:, k]) for k in range(3))
    return x << np.uint64(2) | y << np.uint64(1) | z


def _largest_bucket(key, at):
    """Keys as (key, index) pairs, split at every OVER-th sample."""
    n = key.size
    rank = np.empty(n, dtype=np.int64)
    rank[np.argsort(key, kind="stable")] = np.arange(n)
    cuts = np.sort(rank[at])[OVER::OVER]
    return int(np.diff(np.concatenate([[0], cuts, [n]])).max())


def _lattice(a, b, c):
    g = np.meshgrid(np.arange(a), np.arange(b), np.arange(c), indexing="ij")
    return np.stack(g, -1).reshape(-1, 3).astype(np.float64)


def _clump(n, every):
    pos = np.random.default_rng(every).normal(size=(n, 3))
    pos[::every] *= 1e-3
    return pos


@pytest.mark.parametrize("order", ["lattice 64 64 64", "lattice 128 64 128", "lattice 64 16 256", "lattice 31 67 100",
                                   "clump 1048576 2", "clump 1048576 64", "clump 262144 256", "clump 100003 2",
                                   "sorted 1048576", "random 2097152"])
def test_no_bucket_beyond_the_cap(places, order):
    kind, *a = order.split()
    a = [int(v) for v in a]
    if kind == "lattice":
        pos = _lattice(*a)
    elif kind == "clump":
        pos = _clump(*a)
    else:
        pos = np.random.default_rng(1).normal(size=(a[0], 3))
        if kind == "sorted":
            pos = pos[np.argsort(pos[:, 0])]
    assert _largest_bucket(_keys(pos), places(len(pos))) <= CAP


@pytest.mark.gpu
@pytest.mark.parametrize("n", [20000, 262144])
def test_bucket_beyond_the_cap_is_in_order(places, n):
    from paper_2110_11658_amd.api import Pbh
    print(f"one bucket of nearly {n} keys", flush=True)
    rng = np.random.default_rng(n)
    at = places(n)
    pos = rng.normal(size=(n, 3)) * 1e-3          # a clump that no sample names,
    pos[rng.permutation(n)[: n // 50]] = 1e-4     # with equal keys in it,
    pos[at] = rng.uniform(1.0, 2.0, size=(at.size, 3))   # and every sample far from it
    p = Pbh(0)
    x, m = torch.from_numpy(pos).cuda(), torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    p.build(x, m)
    order, keys, _, _ = p.debug_tree()
    p.close()
    by_caller = np.empty(n, dtype=np.uint64)
    by_caller[order] = keys
    assert _largest_bucket(by_caller, at) > CAP   # (the branch is reached)
    assert np.array_equal(order, np.argsort(by_caller, kind="stable"))

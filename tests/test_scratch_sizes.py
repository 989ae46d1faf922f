"""Scratch that a context keeps is sized for every later build that fits in it.

A build of fewer clusters takes more copies of the group histograms than one of
more: buffers made for 130 clusters serve 128 (and 4, and 1) as well.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2110_11658_amd import ic

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
#include <cstdio>
#include "pbh_internal.hpp"
int main() {
    using namespace pbh;
    for (int64_t made = 1; made <= 1200; ++made)
        for (int64_t used = 1; used <= made; ++used)
            if (kOctaves * used * group_hist_reps((int)used) > group_hist_words(made)) {
                std::printf("made for %lld, used for %lld", (long long)made, (long long)used);
                return 1;
            }
    return 0;
}
"""


def test_group_histograms_fit_every_smaller_count(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if cxx is None or not os.path.isdir(os.path.join(rocm, "include", "hip")):
        pytest.skip("no host compiler or HIP headers")
    src, exe = tmp_path / "sizes.cpp", tmp_path / "sizes"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I",
                    os.path.join(ROOT, "paper_2110_11658_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.gpu
def test_fewer_clusters_on_the_same_context():
    from paper_2110_11658_amd.api import Pbh
    n = 130 * 40
    c = ic.plummer(n, seed=12, masses="kroupa")
    pos, mass = torch.from_numpy(c.pos).cuda(), torch.from_numpy(c.mass).cuda()

    def force(p, k):
        p.build_batched(np.linspace(0, n, k + 1).astype(np.int64), pos, mass)
        return [t.cpu().numpy() for t in p.force_batched([0.01] * k, [0.1] * k, 0.5, 1e-4)]

    kept = Pbh(0, key_bits=18)
    for k in (130, 128, 4, 5, 1):
        print(f"clusters {k}", flush=True)
        fresh = Pbh(0, key_bits=18)
        for a, b in zip(force(kept, k), force(fresh, k)):
            assert np.array_equal(a, b)
        fresh.close()
    kept.close()

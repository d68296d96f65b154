"""LDS that the envs of a pool ask for, from the host's own structures (no GPU
needed): a group of 24x24 1v1 boards leaves room for 32 envs a CU (8 waves a
SIMD) however many envs it has.  A server sizes its launches, and persistent
and two-wave pools theirs, by gen_pool::lds_per_wave."""
import os
import shutil
import subprocess

import pytest

import paper_2606_23348_amd as gen

CSRC = os.path.join(os.path.dirname(os.path.abspath(gen.__file__)), "csrc")
HIPCC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
PROGRAM = r"""
#include <cstdio>
#include "internal.hpp"
int main()
{
    for (int n : {100, 7000, 20000}) {
        std::vector<gen_env_spec> specs((size_t)n);
        for (auto &s : specs) { s = gen_env_spec{}; s.H = 24; s.W = 24; s.mode = GEN_1V1; s.n_players = 2; s.cities_min = 8; s.cities_max = 12; s.min_general_dist = 9; }
        gen_pool *p = nullptr;
        if (gen_pool_create(1, 0, n, specs.data(), nullptr, &p) != GEN_OK) { std::puts(gen_last_error()); return 1; }
        std::printf("%d %u\n", n, p->lds_per_wave);
        gen_pool_destroy(p);
    }
    return 0;
}
"""


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
def test_large_groups_keep_32_envs_a_cu(tmp_path):
    src, exe, lib = tmp_path / "lds.cpp", tmp_path / "lds", os.path.join(os.path.dirname(CSRC), "libgenerals.so")
    src.write_text(PROGRAM)
    subprocess.check_call([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O0", "-w", "-I", CSRC, "-c",
                           "-o", str(exe) + ".o", str(src)])
    subprocess.check_call([HIPCC, "-o", str(exe), str(exe) + ".o", lib, "-Wl,-rpath," + os.path.dirname(lib)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()
    lds = {int(n): int(b) for n, b in zip(out[::2], out[1::2])}
    assert len(lds) == 3
    for n, b in lds.items():
        assert b * 32 <= 160 * 1024, f"{n} envs: {b} bytes an env"

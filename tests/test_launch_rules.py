"""The rules that shape launches (csrc/launch_rules.h), compiled for the host and evaluated over the sizes that contexts accept."""
import ctypes as C
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
#include "launch_rules.h"
extern "C" {
int split_keys(int bf16, int h_kv, int n_keys) { return locret::decode_split_keys(bf16 != 0, h_kv, n_keys); }
int f32_units(int T, int h_kv, int d_R, int64_t room) { return locret::f32_hidden_units(T, h_kv, d_R, room); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "shim.cpp").write_text(SHIM)
    so = d / "shim.so"
    inc = os.path.join(ROOT, "paper_2410_01805_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", inc, str(d / "shim.cpp"), "-o", str(so)], check=True)
    return C.CDLL(str(so))


def test_decode_splits_grow_with_the_cache(rules):
    """Around 700 workgroups on long caches, at every size up to the largest cache a context takes."""
    rng = random.Random(0)
    cases = [(32, 2_900_000), (1024, 131_072), (1024, (1 << 28) - 1), (1, (1 << 28) - 1), (8, 0), (8, 1), (1024, 1)]
    cases += [(rng.randint(1, 1024), int(2 ** rng.uniform(0, 28))) for _ in range(3000)]
    for h_kv, n in cases:
        k = rules.split_keys(1, h_kv, n)
        want = min(65536, h_kv * n // 704)
        assert k % 64 == 0 and max(128, want // 2 - 64) <= k <= max(320, want + 64), (h_kv, n, k)
        k = rules.split_keys(0, h_kv, n)
        assert k % 64 == 0 and max(128, want) <= k <= max(128, want + 64), (h_kv, n, k)


@pytest.mark.parametrize("T,h_kv,d_R,units", [
    (512, 2, 256, 32), (513, 2, 256, 64), (611, 2, 256, 64), (900, 2, 256, 64), (4096, 2, 256, 64), (1, 2, 256, 32),
    (128, 8, 1024, 32), (129, 8, 1024, 64), (200, 8, 1024, 64), (4096, 1, 32, 32), (4097, 1, 32, 64), (4096, 1, 33, 64), (1, 1, 65536, 64),
])
def test_finer_float32_retaining_head_has_one_workgroup_a_cu(rules, T, h_kv, d_R, units):
    f = rules.f32_units
    f.argtypes = [C.c_int] * 3 + [C.c_int64]
    assert f(T, h_kv, d_R, 1 << 20) == units
    partials = -(-d_R // 32) * h_kv * T
    assert f(T, h_kv, d_R, partials) == units and f(T, h_kv, d_R, partials - 1) == 64

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
void score_plan(int T, int h_kv, int K, int d_R, int64_t zpart, int64_t fine, int nt, int split, int* out) {
  const locret::ScorePlan p = locret::plan_score(T, h_kv, K, d_R, zpart, fine, nt, split);
  out[0] = p.mt; out[1] = p.nt; out[2] = p.n_z; out[3] = p.hidden_first;
}
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


def _score_plan(rules, T, h_kv, K, d_R, zpart=None, fine=1 << 20, nt=0, split=-1):
    out = (C.c_int * 4)()
    rules.score_plan.argtypes = [C.c_int] * 4 + [C.c_int64] * 2 + [C.c_int] * 2 + [C.POINTER(C.c_int)]
    rules.score_plan.restype = None
    rules.score_plan(T, h_kv, K, d_R, 4096 * d_R if zpart is None else zpart, fine, nt, split, out)
    return tuple(out)


@pytest.mark.parametrize("T,h_kv,K,d_R,plan", [
    (300, 8, 6144, 1024, (64, 64, 3, 1)),
    (900, 8, 6144, 1024, (64, 64, 1, 1)),
    (1024, 8, 6144, 1024, (64, 64, 1, 0)),
    (611, 8, 6144, 1024, (64, 64, 1, 1)),
    (611, 4, 3072, 1024, (64, 64, 1, 1)),
    (611, 32, 9216, 1024, (64, 64, 1, 1)),
    (900, 8, 6144, 512, (64, 64, 2, 1)),
    (1000, 8, 3072, 512, (64, 64, 2, 0)),
    (1100, 8, 6144, 512, (128, 64, 3, 0)),
    (1300, 8, 6144, 512, (128, 64, 3, 0)),
    (1300, 4, 3072, 512, (64, 64, 1, 1)),
    (900, 8, 6144, 384, (128, 64, 4, 0)),
    (1300, 8, 6144, 384, (128, 64, 3, 0)),
    (1024, 8, 6144, 256, (64, 64, 4, 0)),
    (1024, 2, 768, 128, (128, 64, 1, 0)),
    (1500, 8, 6144, 1024, (128, 64, 1, 0)),
    (4096, 8, 6144, 1024, (128, 128, 1, 0)),
    (512, 8, 6144, 512, (64, 64, 4, 0)),
])
def test_retaining_head_tiles_are_those_that_measured_faster(rules, T, h_kv, K, d_R, plan):
    assert _score_plan(rules, T, h_kv, K, d_R) == plan


def test_retaining_head_plans_are_possible_and_their_order_the_better_one(rules):
    rng = random.Random(1)
    for _ in range(2000):
        T, h_kv, d_R = int(2 ** rng.uniform(0, 13)), rng.choice([1, 2, 4, 8, 16, 24, 32, 64]), 128 * rng.randint(1, 16)
        K, zpart = 64 * rng.randint(3, 200), rng.choice([0, 4096 * d_R])
        mt, nt, n_z, hidden_first = _score_plan(rules, T, h_kv, K, d_R, zpart)
        stages, tt, th = K // 64, -(-T // nt), d_R // mt
        assert n_z == 1 or (n_z * T * d_R <= zpart and (n_z - 1) * -(-stages // n_z) < stages)
        assert mt == 128 or (nt == 64 and tt * th <= 256 and th * h_kv * T <= 1 << 20)
        assert not hidden_first or mt == 64
        if mt == 64 and tt * th >= 64:
            # the tiles that the workgroups of one XCD (every eighth) take, in either order
            seen = lambda n, fast: sum(len({i % fast for i in range(x, n, 8)}) + len({i // fast for i in range(x, n, 8)}) for x in range(8))
            chosen, other = (seen(tt * th, th), seen(tt * th, tt)) if hidden_first else (seen(tt * th, tt), seen(tt * th, th))
            assert chosen <= other * 1.15 + 8, (tt, th, chosen, other)

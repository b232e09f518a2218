"""The GPU tests of the fp32 products reach every kernel that the rule can choose, by the rule itself, on the host: ffn_f32_rule.h is plain
C++; the check is a program around it."""
import os
import subprocess

import test_gpu_parity as G

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KERNELS = ("few rows", "parts, 64 weight rows", "parts, 128 weight rows")

PROGRAM = r"""
#include <cstdio>
#include "ffn_f32_rule.h"
int main() {
    long long glu, A, K, N, E;
    while (std::scanf("%lld %lld %lld %lld %lld", &glu, &A, &K, &N, &E) == 5) std::printf("%d\n", moe_f32_kernel(glu != 0, A, K, N, E));
}
"""


def kernels(tmp_path, products):
    """[(swiglu, A, K, N, E)] -> the kernel of each"""
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2506_12417_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, p)) for p in products), capture_output=True, text=True, check=True)
    return [KERNELS[int(v)] for v in out.stdout.split()]


def first_products(cases):
    return [(int(act == "swiglu"), sum(rows), d, (2 if act == "swiglu" else 1) * F, len(rows)) for rows, d, F, act in cases]


def test_the_products_of_the_gpu_tests_take_every_kernel(tmp_path):
    cases = [(rows, d, F, act) for rows, _, d, F, act, _ in G.F32_CASES + G.F32_FEW_CASES]
    firsts = kernels(tmp_path, first_products(cases))
    seconds = kernels(tmp_path, [(0, sum(rows), F, d, len(rows)) for rows, d, F, act in cases])
    assert {(act, got) for (_, _, _, act), got in zip(cases, firsts)} == {(act, k) for act in ("relu", "swiglu") for k in KERNELS}
    assert set(seconds) == set(KERNELS)


def test_the_extreme_values_of_the_gpu_tests_meet_every_kernel(tmp_path):
    every = {(act, k) for act in ("relu", "swiglu") for k in KERNELS}
    extreme = kernels(tmp_path, first_products(G.F32_EXTREME_CASES))
    assert {(c[3], got) for c, got in zip(G.F32_EXTREME_CASES, extreme)} == every
    ranges = kernels(tmp_path, first_products(G.F32_RANGE_SHAPES))
    assert {(c[3], got) for c, got in zip(G.F32_RANGE_SHAPES, ranges)} == every - {("swiglu", KERNELS[0])}
    assert set(kernels(tmp_path, first_products([c + ("relu",) for c in G.F32_SINGLE_TERM_SHAPES]))) == set(KERNELS)

"""The sizes of tests/test_gpu_layer_shapes.py reach every kernel form that the
planners choose (CPU).

tests/host/plan_check.cpp compiles the library's own planner header and answers
which projection tile or attention form a size takes.  A sweep over the sizes the
library accepts finds the choices that occur; each has to occur among the tested
sizes too, with a remainder where the kernel has a code path for one.
"""
import os
import random
import shutil
import subprocess

import pytest

import test_gpu_layer_shapes as shapes

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++") or shutil.which("clang++")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if CXX is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("plan") / "plan_check")
    subprocess.run([CXX, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2609_34608_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "plan_check.cpp"), "-o", exe], check=True, timeout=120)

    def answers(lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=120)
        assert r.returncode == 0
        out = [x.split() for x in r.stdout.splitlines()]
        assert len(out) == len(lines)
        return out

    return answers


def _table(ask, name):
    """Every entry of a planner's cost table."""
    return set(ask([f"table {name}"])[0])


def _projections(ask, dtype, sizes, remainders):
    """{(tile, epilogue)} of the four projections of (B, T, D, dh, F) sizes; with
    remainders, only those whose last row tile is not full and, of 256 columns,
    whose last column tile is not full."""
    lines = []
    for B, T, D, dh, F in sizes:
        lines += [f"{dtype} {B * T} {n} {k} {int(qkv)}" for n, k, qkv in
                  ((3 * D, D, True), (D, D, False), (F, D, False), (D, F, False))]
    found = set()
    for i, tile in enumerate(ask(lines)):
        B, T, D, dh, F = sizes[i // 4]
        N, epi = ((3 * D, f"qkv{dh}"), (D, "gated"), (F, "gelu"), (D, "gated"))[i % 4]
        bm, bn, _ = map(int, tile[0].split("x"))
        if remainders and (B * T % bm == 0 or (bn == 256 and N % bn == 0)):
            continue
        found.add((tile[0], epi))
    return found


def _sweep(n, fp32):
    rng = random.Random(17)
    out = []
    while len(out) < n:
        B, D = rng.choice([1, 1, 1, 2, 3, 4, 8, 16]), 64 * rng.randint(1, 16 if fp32 else 32)
        T = int(3 * 1000 ** rng.random()) if rng.random() < 0.5 else rng.randint(100, 12000)
        F = 128 * rng.randint(1, max(1, 4 * D // 128))
        if B * T <= 16000:
            out.append((B, T, D, rng.choice([32, 64]) if fp32 else 64, F))
    return out


def test_bf16_projection_tiles(ask):
    tested = [(B, T, D, 64, F) for B, T, D, F in shapes.BF16_LAYERS + shapes.BF16_TILES]
    tested += [(B, T, D, 64, 2 * D) for B, T, D in shapes.BF16_ATTENTION]
    chosen = _projections(ask, "bf16", _sweep(20000, False), False)
    assert {t for t, _ in chosen} == _table(ask, "bf16")
    missing = chosen - _projections(ask, "bf16", tested, True)
    assert not missing, missing


def test_float32_projection_tiles(ask):
    chosen = _projections(ask, "fp32", _sweep(20000, True), False)
    assert {t for t, _ in chosen} == _table(ask, "fp32")
    missing = chosen - _projections(ask, "fp32", [s[:5] for s in shapes.FP32_LAYERS], True)
    assert not missing, missing


@pytest.mark.parametrize("kind", ["bounded", "running"])
def test_bf16_attention_forms(ask, kind):
    def forms(sizes, remainders):
        found = set()
        for (B, T, D), (form,) in zip(sizes, ask([f"{kind} {T} {B * D // 64}" for B, T, D in sizes])):
            qt, nw = map(int, form.split(":")[1].split("x"))
            # queries of the last block: some, and so few that a wave gets none
            if not remainders or 0 < T % (16 * qt * nw) <= 16 * qt * (nw - 1):
                found.add(form)
        return found
    chosen = forms([s[:3] for s in _sweep(20000, False)], False)
    assert chosen == _table(ask, kind)
    missing = chosen - forms(shapes.BF16_ATTENTION, True)
    assert not missing, missing


def test_key_split_of_one_key_tile(ask):
    sizes = [(B, T, D) for B, T, D in shapes.BF16_ATTENTION if T <= 64]
    split = max(_table(ask, "bounded"))  # form 4: two wave groups split the keys
    assert split.startswith("4:")
    assert [split] in ask([f"bounded {T} {B * D // 64}" for B, T, D in sizes])


def test_float32_attention_forms(ask):
    sizes = [s[:4] for s in shapes.FP32_LAYERS if s[1] % 16]
    got = {(f[0], dh) for (B, T, D, dh), f in
           zip(sizes, ask([f"attn_fp32 {T} {B * D // dh}" for B, T, D, dh in sizes]))}
    assert got == {(f, dh) for f in "012" for dh in (32, 64)}

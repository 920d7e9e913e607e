"""The device tree compiler's bottom-up pass through blocks and walks, and its emission by a thread per node, run on the CPU:
the host compiler's programs byte for byte.  tests/csrc/devcompile_block_emu.cpp runs the steps that the kernels run
(paper_2205_03251_amd/csrc/devcompile_core.h) in random interleavings, in blocks small enough for most trees to leave theirs;
a mistake planted in a copy of each step is found."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import gen
from test_devcompile_emu import comb, complete, random_points

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2205_03251_amd", "csrc")


def build(folder, change=None):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    src = os.path.join(HERE, "csrc", "devcompile_block_emu.cpp")
    if change:
        for name in os.listdir(CSRC):
            if name.endswith((".h", ".cpp")):
                shutil.copy(os.path.join(CSRC, name), folder)
        core = open(os.path.join(CSRC, "devcompile_core.h")).read()
        assert core.count(change[0]) == 1, change
        open(os.path.join(folder, "devcompile_core.h"), "w").write(core.replace(*change))
        text = open(src).read().replace("../../paper_2205_03251_amd/csrc/devcompile_core.h", "devcompile_core.h")
        src = os.path.join(folder, "emu.cpp")
        open(src, "w").write(text)
    exe = os.path.join(folder, "block_emu")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-o", exe, src, os.path.join(CSRC, "prep.cpp")], check=True)
    return exe


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("block_emu")))


def run(exe, pop, chunk_nodes, span, index_min=0, points=None, seed=1, check=True):
    flat = [(t, c) for t, p in enumerate(points or []) for c in p]
    head = [pop.vtype, pop.n_inputs, chunk_nodes, index_min, pop.n_trees, seed, span, len(flat)]
    text = "\n".join([" ".join(map(str, head)), " ".join(map(str, pop.offsets.tolist())), " ".join(map(str, pop.ops.tolist())),
                      " ".join(f"{t} {c}" for t, c in flat)]) + "\n"
    r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=600)
    if not check:
        return r.returncode == 0
    assert r.returncode == 0, r.stdout + r.stderr
    f = r.stdout.split()
    return dict(zip(f[1::2], map(int, f[2::2])))


@pytest.mark.parametrize("span", [1, 7, 64, 4096])
@pytest.mark.parametrize("vtype,n_terms,chunk_nodes", [(gen.VT_F32, 1, 64), (gen.VT_F32, 3, 1024), (gen.VT_BOOL, 6, 256)])
def test_sized_trees(emu, span, vtype, n_terms, chunk_nodes):
    pop = gen.sized_population(17 + span, 24, 1, 12001, n_terms=n_terms, vtype=vtype)
    got = run(emu, pop, chunk_nodes, span, 512, random_points(8, pop, 2), seed=span)
    assert got["chunks"] > pop.n_trees and got["listed"] > 0
    assert span > 64 or got["between"] > 100


@pytest.mark.parametrize("span", [5, 100, 4096])
def test_combs_complete_trees_and_single_nodes(emu, span):
    trees = [comb(3000, True, seed=1), np.array([0], np.uint8), comb(2999, False, seed=2), complete(12, seed=3),
             np.array([0x81, 0, 0], np.uint8), np.array([0], np.uint8), complete(6, seed=4)]
    pop = gen.pack(trees, gen.VT_F32, 1)
    pts = [[0, 5, 2999, 6000], [0], [1, 5997, 3000], [17], [0, 1, 2], [], [3]]
    for c in (2, 16, 1024, 8192):
        run(emu, pop, c, span, 64, pts, seed=c)


def test_many_tiny_trees(emu):
    pop = gen.sized_population(4, 800, 1, 9)
    for span in (3, 16, 4096):
        run(emu, pop, 512, span)


MISTAKES = {
    "an outside parent taken for the root": ("    if (p == kDcOutside) return -2;\n", "    if (p == kDcOutside) return -1;\n"),
    "operands exchanged in a block": ("dc_unpack(left ? *w : other), dc_unpack(left ? other : *w));\n    b.word[p]",
                                      "dc_unpack(left ? other : *w), dc_unpack(left ? *w : other));\n    b.word[p]"),
    "a block's cut lost": ("    if (o.cut_kids & 1) Mem::fetch_or(b.word + l, (uint32_t)kDcCut);\n", ""),
    "the left word in the wrong half": ("((uint32_t*)q.slot64)[2 * (base + p)] = *w;", "((uint32_t*)q.slot64)[2 * (base + p) + 1] = *w;"),
    "the atomic's answer ignored": ("        other = left ? (uint32_t)(old >> 32) : (uint32_t)old;\n        if (other == 0) return -1;",
                                    "        (void)old;\n        return -1;"),
    "a walk's own parent not taken over": ("    *p = pp;\n", ""),
    "the second operand one slot too low": ("    *by = ((uint32_t)w << kDcSlotBits) + 1u;\n", "    *by = ((uint32_t)w << kDcSlotBits);\n"),
    "a chunk's id not given back": ("    if (end < n) Mem::add(step + end, 0u - by);\n", ""),
    "the second operand's LOAD first": ("    return pg * 2 + (two && ", "    return pg * 2 - (two && "),
    "a STORE left out": ("        code[pos + 1] = store;\n", ""),
}


@pytest.mark.parametrize("what", sorted(MISTAKES))
def test_mistakes_are_found(what, tmp_path):
    exe = build(str(tmp_path), MISTAKES[what])
    found = []
    for seed in (1, 2, 3):
        pop = gen.sized_population(30 + seed, 12, 101, 4001, n_terms=2)
        found += [not run(exe, pop, c, span, 64, random_points(seed, pop, 2), seed, check=False)
                  for c, span in ((32, 24), (256, 100), (128, 4096))]
    assert any(found), what

"""The host grouping of chunks that share lists (csrc/ppcg_groups.hpp), compiled alone: every chunk's entries lie
inside its representative's, whatever the hashes."""

import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2105_06176_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "ppcg_groups.hpp"
int main()
{
    int nc;
    long long cap;
    if (scanf("%d %lld", &nc, &cap) != 2)
        return 1;
    std::vector<int64_t> cptr(1, 0);
    std::vector<unsigned long long> hash;
    for (int c = 0; c < nc; ++c) {
        int len;
        unsigned long long a, b;
        if (scanf("%d %llu %llu", &len, &a, &b) != 3)
            return 1;
        cptr.push_back(cptr.back() + 64 * (int64_t)len);
        hash.push_back(a);
        hash.push_back(b);
    }
    ppcg::ChunkGroups g;
    const bool ok = ppcg::group_chunks(nc, 64, cptr.data(), hash.data(), cap, &g);
    printf("%d %lld %lld %d\n", (int)ok, (long long)g.nlist, (long long)g.nmask, g.longest);
    for (const auto &c : g.chunk)
        printf("c %d %d %d\n", c.list, c.mask, c.len);
    for (const auto &i : g.items)
        printf("i %d %d %d\n", i.chunk, i.dst, i.masks);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("groups")
    (d / "m.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(d / "m"), str(d / "m.cpp")], check=True)
    return str(d / "m")


def group(program, chunks, cap=1 << 40):
    text = f"{len(chunks)} {cap}\n" + "\n".join("%d %d %d" % c for c in chunks)
    out = subprocess.run([program], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    ok, nlist, nmask, longest = map(int, out[0].split())
    got = {k: [tuple(map(int, ln.split()[1:])) for ln in out[1:] if ln.startswith(k)] for k in "ci"}
    return bool(ok), nlist, nmask, longest, got["c"], got["i"]


def check(chunks, res):
    ok, nlist, nmask, longest, cs, items = res
    assert ok and longest == max(c[0] for c in chunks)
    reps = ({d: chunks[c] for c, d, m in items if m == 0}, {d: chunks[c] for c, d, m in items if m == 1})
    for (length, hl, hm), (lst, msk, n) in zip(chunks, cs):
        assert n == length
        assert reps[0][lst][0] == length and reps[0][lst][1] == hl and lst + length <= nlist
        assert reps[1][msk][0] == length and reps[1][msk][2] == hm and msk + length <= nmask


def test_equal_hashes_of_other_lengths_do_not_share(program):
    chunks = [(3, 7, 9), (1000, 7, 9), (3, 7, 9), (5, 7, 8)]
    res = group(program, chunks)
    check(chunks, res)
    assert res[1:3] == (1008, 1008) and len(res[5]) == 6


@pytest.mark.parametrize("seed", range(3))
def test_random_hashes(program, seed):
    rng = random.Random(seed)
    chunks = [(rng.randint(1, 6), rng.randint(0, 4), rng.randint(0, 4)) for _ in range(300)]
    check(chunks, group(program, chunks))


def test_lists_past_the_cap_are_refused(program):
    chunks = [(10, k, 1) for k in range(20)]
    need = 12 * 200 + 8 * 10
    assert group(program, chunks, need)[0] and not group(program, chunks, need - 1)[0]

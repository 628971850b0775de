"""The memory pool of a server's requests (csrc/ppcg_pool.hip) on the host, over a device memory that only counts."""

import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2105_06176_amd", "csrc")

# Commands: L limit, C capacity of the device, N name bytes (take), F name (give).  After each: result, bytes of the
# device in use, most of them so far, bytes counted for the thread, stream synchronizations.
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <string>
#include "ppcg_pool.hpp"
static size_t used, most, capacity = (size_t)-1;
static int syncs;
static std::map<void *, size_t> blocks;
extern "C" {
hipError_t hipMalloc(void **p, size_t n)
{
    if (n > capacity || used > capacity - n)
        return hipErrorOutOfMemory;
    *p = malloc(1);
    blocks[*p] = n;
    used += n;
    most = used > most ? used : most;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    used -= blocks.at(p);
    blocks.erase(p);
    free(p);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { ++syncs; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}
int main()
{
    {
        ppcg::DevPool pool;
        std::map<int, void *> held;
        ppcg::DevPool::use().pool = &pool;
        char op;
        int name;
        size_t n;
        while (scanf(" %c", &op) == 1) {
            int rc = 0;
            if (op == 'L' && scanf("%zu", &n) == 1)
                pool.set_limit(n);
            if (op == 'C' && scanf("%zu", &n) == 1)
                capacity = n;
            if (op == 'S' && scanf("%zu", &n) == 1)
                ppcg::DevPool::use().stream = (hipStream_t)n;
            if (op == 'N' && scanf("%d %zu", &name, &n) == 2) {
                void *p = nullptr;
                rc = pool.take(&p, n);
                if (rc == 0) {
                    if (blocks.at(p) < n)
                        return 2;
                    held[name] = p;
                }
            }
            if (op == 'F' && scanf("%d", &name) == 1) {
                if (!ppcg::DevPool::give(held.at(name)))
                    return 3;
                held.erase(name);
            }
            printf("%d %zu %zu %lld %d\n", rc, used, most, (long long)ppcg::DevPool::use().bytes, syncs);
        }
    }
    printf("%zu\n", used);
    return ppcg::DevPool::give(&used) ? 4 : 0;  // no pool's
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("pool")
    (d / "m.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, "-o",
                    str(d / "m"), "-x", "c++", str(d / "m.cpp"), os.path.join(CSRC, "ppcg_pool.hip"), "-lpthread"],
                   check=True)
    return str(d / "m")


def run(program, script):
    r = subprocess.run([program], input=script, capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr)
    lines = r.stdout.split("\n")
    steps = [tuple(map(int, ln.split())) for ln in lines[:-2]]
    return steps, int(lines[-2])


M = 1 << 20


def test_idle_blocks_count_against_the_limit(program):
    # six blocks of 4 MiB given back, then as many bytes in other sizes
    script = f"L {30 * M}\n" + "".join(f"N {k} {4 * M}\n" for k in range(6)) + "".join(f"F {k}\n" for k in range(6))
    script += "".join(f"N {k} {7 * M}\n" for k in range(4))
    steps, left = run(program, script)
    assert steps[-1][0] == 0 and steps[-1][2] <= 30 * M and left == 28 * M  # (the four are still out)


def test_sizes_are_exact_where_rounding_would_pass_the_limit(program):
    steps, _ = run(program, f"L {10 * M}\nN 0 {5 * M + 1}\nN 1 {4 * M + 5}\n")
    assert steps[-1][1] <= 10 * M + 256 and steps[1][1] == 6 * M


def test_large_blocks_are_counted_and_tried_again(program):
    script = f"C {100 * M}\nN 0 {30 * M}\nN 1 {30 * M}\nF 0\nF 1\nN 2 {90 * M}\nF 2\n"
    steps, left = run(program, script)
    assert all(s[0] == 0 for s in steps) and steps[-1][1] == 0 and left == 0  # a block above 32 MiB is not kept
    assert run(program, f"C {100 * M}\nN 0 {101 * M}\n")[0][-1][:2] == (2, 0)


def test_reuse_and_what_is_kept(program):
    steps, left = run(program, "N 0 100000\nF 0\nN 1 99000\nF 1\n" + "".join(f"N {k} {16 * M}\n" for k in range(20)) +
                      "".join(f"F {k}\n" for k in range(20)))
    assert steps[2][1] == steps[0][1] == 114688 and steps[1][3] == 0 and steps[2][3] == 114688
    assert 240 * M <= steps[-1][1] <= 256 * M and left == 0


def test_the_threads_stream_is_synchronized(program):
    steps, _ = run(program, "N 0 1000\nF 0\nS 8\nN 0 1000\nF 0\n")
    assert [s[4] for s in steps] == [0, 0, 0, 0, 1]


@pytest.mark.parametrize("seed", range(4))
def test_random_sequences_stay_within_the_limit(program, seed):
    rng = random.Random(seed)
    limit, held, out, script, name = 64 * M, {}, 0, f"L {64 * M}\n", 0
    for _ in range(400):
        n = int(2 ** rng.uniform(5, 25))
        if held and (rng.random() < 0.45 or out + n > limit - 4096):
            k = rng.choice(sorted(held))
            out -= held.pop(k)
            script += f"F {k}\n"
        else:
            held[name] = max(n, 256)
            out += held[name]
            script += f"N {name} {n}\n"
            name += 1
    for k in held:
        script += f"F {k}\n"
    steps, left = run(program, script)
    assert all(s[0] == 0 for s in steps) and left == 0
    # rounded sizes in use come first to the limit, exact ones after it
    assert steps[-1][2] <= limit * 5 // 4 and all(s[1] <= limit for s in steps[-len(held):])

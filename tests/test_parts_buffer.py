"""The handle's buffer for products cut along k (csrc/parts_buffer.h), compiled for the
host with an allocator that counts, and refuses from a given size on: memory is asked for
only where the buffer does not suffice, an outgrown buffer is not freed under calls and
graphs that may use it, and a refused size is not asked for again until the workspace moves."""
import os
import subprocess

import pytest

HARNESS = r"""
#include <cassert>
#include <cstdio>
#include <set>
#include "parts_buffer.h"
static std::set<void *> live;
static size_t limit, last;
static int asked;
static char arena[64];
static void *take(size_t size) {
    ++asked;
    last = size;
    if (size > limit) return nullptr;
    void *p = arena + asked;
    live.insert(p);
    return p;
}
static void give(void *p) { assert(live.erase(p) == 1); }
#define CHECK(x) if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; }
int main() {
    ozc::PartsBuffer b;
    const size_t M = (size_t)1 << 20;
    limit = 40 * M;
    CHECK(!b.covers(1));
    void *p = b.get(5 * M, take);
    CHECK(p && asked == 1 && b.covers(5 * M));
    CHECK(b.get(3 * M, take) == p && b.get(5 * M, take) == p && asked == 1);
    void *q = b.get(6 * M, take);                       // grows to twice the size
    CHECK(q && q != p && asked == 2 && last == 10 * M && live.size() == 2);  // p is kept
    CHECK(b.get(1, take) == q && b.get(10 * M, take) == q && asked == 2);
    CHECK(!b.get(41 * M, take) && asked == 3);          // refused: what there is stays
    CHECK(!b.get(41 * M, take) && !b.get(99 * M, take) && asked == 3);
    CHECK(b.get(10 * M, take) == q && live.size() == 2);
    CHECK(b.get(30 * M, take) && asked == 4 && live.size() == 3);
    b.release(give);                                    // the workspace moves
    CHECK(live.empty() && !b.covers(1));
    limit = 50 * M;
    CHECK(b.get(41 * M, take) && asked == 5);
    limit = SIZE_MAX;
    for (int e = 26; e < 64; ++e) CHECK(b.get((size_t)1 << e, take));
    b.release(give);
    CHECK(live.empty());
    b.release(give);
    puts("ok");
}
"""


def test_buffer(tmp_path):
    csrc = os.path.join(os.path.dirname(__file__), "..", "paper_2512_08321_amd", "csrc")
    (tmp_path / "h.cpp").write_text(HARNESS)
    exe = str(tmp_path / "h")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-fsanitize=undefined,bounds",
                    "-fno-sanitize-recover=all", "-I" + csrc, str(tmp_path / "h.cpp"), "-o", exe], check=True)
    assert subprocess.run([exe], capture_output=True, text=True, check=False).stdout == "ok\n"


def _operands(m, n, k, seed):
    import torch

    g = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn(s, dtype=torch.complex128, device="cuda", generator=g) for s in ((k, m), (n, k))]


@pytest.mark.gpu
def test_workspace_stays_under_a_captured_graph():
    """A graph holds the workspace's address: a later call that it suffices for, but for the
    parts' planes, leaves it where it is; the same call in a capture takes whole products
    while there is no buffer for the parts, and the parts once there is."""
    import torch

    import paper_2512_08321_amd as ozc

    h = ozc.Handle(0, num_moduli=14)
    try:
        # whole products; products cut along k, for which that workspace just suffices
        big, cut = (1000, 900, 1100), (64, 96, 6400)
        need = {big: h.workspace_size("N", "N", *big)}
        while h.workspace_size("N", "N", *cut[:2], cut[2] + 64) <= need[big]:
            cut = (*cut[:2], cut[2] + 64)
        need[cut] = h.workspace_size("N", "N", *cut)
        ops = {s: _operands(*s, 7 + i) for i, s in enumerate((big, cut))}

        def call(s):
            (m, n, k), (A, B) = s, ops[s]
            C = torch.zeros((n, m), dtype=torch.complex128, device="cuda")
            h.zgemm("N", "N", m, n, k, 1.0, A, m, B, k, 0.0, C, m)
            return C

        def capture(s):
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                C = call(s)
            return graph, C

        print("parts buffer: warm-up", flush=True)
        want = {big: call(big).clone()}
        assert h.last_info()["workspace"] == need[big]
        torch.cuda.synchronize()
        print("parts buffer: capture", flush=True)
        graphs = [(big, *capture(big)), (cut, *capture(cut))]
        assert h.last_info()["workspace"] == need[cut]   # nothing allocated in the capture
        want[cut] = call(cut).clone()
        assert h.last_info()["workspace"] > need[big]    # the parts, in a buffer of their own
        torch.cuda.synchronize()
        graphs.append((cut, *capture(cut)))
        assert h.last_info()["workspace"] > need[cut]
        for _ in range(3):
            for s, graph, C in graphs:
                C.zero_()
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(C, want[s])
            call(cut)
            call(big)
    finally:
        torch.cuda.synchronize()
        h.close()

"""The pool of captured rounds, compiled for the host: at its limit it makes room
once and keeps what is captured next, so a round's pair is there for the rounds
after it; a changed signature drops every pair, each graph destroyed once."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROBE = r"""
#include "round_graphs.h"
#include <cstdio>
#include <set>
using Pool = hbsjd::RoundGraphPool<int, int>;

int main() {
    std::set<int> live;
    int next = 1, captures = 0, twice = 0;
    auto destroy = [&](int e) { twice += live.erase(e) != 1; };
    Pool pool(3);
    // one round under row bound `bound`, whose products take the kernels `plan`
    auto round = [&](uint64_t sig, int bound, int plan) {
        pool.match({sig}, destroy);
        auto* p = pool.find(bound, [&](const std::vector<int>& x) { return x[0] == plan; });
        if (!p) {
            if (pool.full()) pool.drop(destroy);
            Pool::Pair g;
            g.plan = {plan};
            g.bound = bound;
            for (int& e : g.exec) live.insert(e = next++);
            p = pool.add(g);
            ++captures;
        }
        return p->exec[0];
    };
    // five plans, four rounds each, as the row bound falls
    for (int plan = 5; plan > 0; --plan)
        for (int r = 0; r < 4; ++r) round(7, 10 * plan - r, plan);
    printf("falling %d %zu\n", captures, live.size());
    captures = 0;
    round(7, 11, 1);                      // above the bound its pair was captured under
    printf("above %d\n", captures);
    captures = 0;
    for (int r = 0; r < 3; ++r) round(8, 20, 2);   // another signature
    printf("signature %d %zu\n", captures, live.size());
    pool.drop(destroy);
    printf("end %zu %d\n", live.size(), twice);
}
"""


def test_pool_of_captured_rounds(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    src, exe = tmp_path / "pool.cpp", tmp_path / "pool"
    src.write_text(PROBE)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2608_18183_amd", "csrc"), str(src), "-o", str(exe)])
    out = subprocess.check_output([str(exe)], text=True).split("\n")
    # five captures; the fourth made room, so the last two pairs are live
    assert out[:4] == ["falling 5 4", "above 1", "signature 1 2", "end 0 0"]

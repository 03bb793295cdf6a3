"""The scratch arena's policy (csrc/arena.h), compiled with g++ over a card of limited room: a call that can run in fewer
groups of steps does not ask again for what the card has refused, so a program on a full card keeps its arena and pays
one refusal, not a wait, a free and two allocations a call.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_12378_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "arena.h"

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

struct Card {
    size_t room, used = 0, held = 0;
    int allocations = 0, refusals = 0, releases = 0;
    bool release(void *) { releases++; used -= held; held = 0; return true; }
    void *allocate(size_t n)
    {
        if (used + n > room) { refusals++; return nullptr; }
        allocations++;
        used += held = n;
        return this;
    }
};

static uint32_t call(Arena &a, Card &c)    // eight groups of 1000 bytes beside 1000
{
    return most_groups(a, 8u, [](uint32_t g) { return (size_t)1000 * (g + 1); },
                       [&](size_t n) { return a.take(n, c) == Arena::OK; });
}

int main()
{
    Arena a;
    Card c{4000};
    CHECK(call(a, c) == 2 && c.refusals == 2 && c.allocations == 1);    // 9000 and 5000 bytes refused, 3000 taken
    for (int i = 0; i < 3; i++) CHECK(call(a, c) == 2);
    CHECK(c.refusals == 2 && c.allocations == 1 && c.releases == 0);    // as it was: nothing asked, nothing dropped
    CHECK(a.take(2000, c) == Arena::OK && c.releases == 0);             // other calls still find the arena
    CHECK(a.take(3500, c) == Arena::OK && c.releases == 1 && c.refusals == 2);   // and may grow it below the refusal
    c.room = 20000;                                                     // the program frees memory
    CHECK(call(a, c) == 2);
    CHECK(a.take(6000, c) == Arena::OK);                                // a call that needs as much finds out
    CHECK(call(a, c) == 8 && c.refusals == 2);
    a.set(nullptr, 0);                                                  // or the arena given back
    c.used = c.held = 0;
    c.room = 2500;
    CHECK(call(a, c) == 1 && call(a, c) == 1 && c.refusals == 5);
    a.set(nullptr, 0);
    c.used = c.held = 0;
    c.room = 500;
    CHECK(call(a, c) == 0 && a.base == nullptr && a.bytes == 0);
    Card w{0};
    a.set(&w, 5000);                                                    // a caller's workspace: four groups fit
    CHECK(call(a, w) == 4 && w.refusals == 0 && a.take(5001, w) == Arena::TOO_SMALL && a.base == &w);
    std::puts("ok");
    return 0;
}
"""


def test_refused_sizes_are_not_asked_for_again(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src = tmp_path / "arena.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "arena")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, str(src), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout

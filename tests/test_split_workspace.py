"""The bookkeeping of the streams' split workspaces, compiled for the host alone
with an allocator that refuses."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "split_workspace.hpp"

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
    int calls = 0, memory = 0, live = 0, freed = 0;
    auto refuse = [&] { ++calls; return (void *)nullptr; };
    auto grant = [&] { ++calls; return (void *)&memory; };
    oc::SplitWorkspace w, x;
    // no memory at the first call: never asked for again, also once there is some
    CHECK(w.get(live, refuse) == nullptr && w.get(live, refuse) == nullptr && w.get(live, grant) == nullptr && calls == 1);
    // memory at the first call: the same workspace ever after
    calls = 0;
    CHECK(x.get(live, grant) == &memory && x.get(live, refuse) == &memory && calls == 1);
    // no more than MAX_SPLIT_WORKSPACES at a time; one given back makes room
    oc::SplitWorkspace many[oc::MAX_SPLIT_WORKSPACES], y, z;
    for (int i = 0; i + 1 < oc::MAX_SPLIT_WORKSPACES; ++i) CHECK(many[i].get(live, grant) == &memory);
    CHECK(live == oc::MAX_SPLIT_WORKSPACES && y.get(live, grant) == nullptr);
    auto release = [&](void *p) { freed += p == &memory; };
    x.give_back(live, release);
    w.give_back(live, release);
    CHECK(freed == 1 && live == oc::MAX_SPLIT_WORKSPACES - 1);
    CHECK(z.get(live, grant) == &memory && y.get(live, grant) == nullptr && live == oc::MAX_SPLIT_WORKSPACES);
    // a capture's own: not the stream's, not the capture before's; asked for once
    live = 0;
    calls = 0;
    int other = 0;
    oc::SplitWorkspace c;
    CHECK(c.get(live, grant) == &memory && calls == 1);
    auto second = [&] { ++calls; return (void *)&other; };
    CHECK(c.get_captured(live, 0, second) == &other && c.get_captured(live, 0, grant) == &other && calls == 2);
    CHECK(c.get_captured(live, 7, refuse) == nullptr && c.get_captured(live, 7, grant) == nullptr && calls == 3);
    CHECK(c.get_captured(live, 8, grant) == &memory && live == 3 && c.get(live, refuse) == &memory && calls == 4);
    live = oc::MAX_SPLIT_WORKSPACES;
    CHECK(c.get_captured(live, 9, grant) == nullptr && calls == 4);
    return 0;
}
"""


def test_workspaces_are_asked_for_once_and_bounded(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2605_22850_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout

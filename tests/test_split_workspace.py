"""The bookkeeping of a stream's split workspace, compiled for the host alone
with an allocator that refuses."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "split_workspace.hpp"

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
    int calls = 0, memory = 0;
    auto refuse = [&] { ++calls; return (void *)nullptr; };
    auto grant = [&] { ++calls; return (void *)&memory; };
    oc::SplitWorkspace w, x;
    // no memory at the first call: never asked for again, also once there is some
    CHECK(w.get(refuse) == nullptr && w.get(refuse) == nullptr && w.get(grant) == nullptr && calls == 1);
    // memory at the first call: the same workspace ever after
    calls = 0;
    CHECK(x.get(grant) == &memory && x.get(refuse) == &memory && calls == 1);
    return 0;
}
"""


def test_workspace_is_asked_for_once(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2605_22850_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout

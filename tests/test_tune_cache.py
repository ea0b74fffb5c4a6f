"""The tuning cache under threads (CPU): every operator apply looks its depth up while
another thread may be tuning another mesh, so lookups, insertions, the first load of the
file and a save overlap.  The cache is host C++; a small program over it runs under the
thread sanitizer, which ends it with an error at the first unlocked access."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2103_00081_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "tune.h"

int main()
{
    hts::TuneCache c;
    std::vector<std::thread> t;
    for (int k = 0; k < 4; k++)                       // applies, the first of which loads the file
        t.emplace_back([&c] {
            for (int i = 0; i < 300; i++)
                if (c.get(4, 1, 0, 129, 129, 65) != 10) std::printf("lost\n");
        });
    t.emplace_back([&c] {                             // autotune of other meshes
        for (int i = 0; i < 300; i++) c.set(5, 0, 1, i + 2, 33, 17, i % 7 + 1);
        c.save();
    });
    for (auto &x : t) x.join();
    for (int i = 0; i < 300; i++)
        if (c.get(5, 0, 1, i + 2, 33, 17) != i % 7 + 1) std::printf("lost\n");
    std::printf("done\n");
}
"""


def test_lookups_while_another_mesh_is_tuned(tmp_path):
    src, exe, cache = (str(tmp_path / f) for f in ("main.cpp", "main", "tune.json"))
    with open(src, "w") as f:
        f.write(PROGRAM)
    with open(cache, "w") as f:
        f.write('{\n  "q4_f1_fp64_129x129x65": 10\n}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-I", CSRC, src, "-o", exe, "-pthread"], check=True)
    env = dict(os.environ, HTS_TUNE_CACHE=cache, TSAN_OPTIONS="halt_on_error=1 exitcode=66")
    r = subprocess.run([exe], env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    if "unexpected memory mapping" in r.stdout:      # its shadow does not fit this kernel's address layout
        pytest.skip("the thread sanitizer cannot run here")
    assert r.returncode == 0 and r.stdout.split() == ["done"], r.stdout[-2000:]
    with open(cache) as f:
        text = f.read()
    assert '"q4_f1_fp64_129x129x65": 10' in text and text.count("q5_f0_fp32") == 300

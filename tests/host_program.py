"""Runs host code of the library's headers (plans, rules, buffer sizes: no device is touched) as a small program."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PRELUDE = """
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>
#include "include/seedinf.h"
#include "paper_1910_06591_amd/csrc/plan.h"
#include "paper_1910_06591_amd/csrc/bf16_path.h"
using namespace seedinf;

// the plan of a ResNet on h x w x c frames with these sections
static Plan resnet(int h, int w, int c, const std::vector<int>& sections)
{
    seed_arch_t a{};
    a.struct_size = sizeof a; a.obs_h = h; a.obs_w = w; a.obs_c = c;
    a.torso = SEED_TORSO_RESNET; a.n_sections = (int)sections.size();
    for (size_t i = 0; i < sections.size(); ++i) a.section_ch[i] = sections[i];
    a.fc_units = 16; a.num_actions = 2; a.head = SEED_HEAD_POLICY_VALUE; a.select = SEED_SELECT_GREEDY;
    a.precision = SEED_PRECISION_BF16; a.max_batch = 1;
    Plan p;
    std::string err;
    if (make_plan(&a, p, err) != SEED_OK) { fprintf(stderr, "%s\\n", err.c_str()); exit(1); }
    return p;
}
"""


def build(tmp_path, main):
    """Compiles the prelude and `main` (C++ with a main function) for the host only; returns a function that runs it on
    lines of text and returns its output lines."""
    src, obj, exe = (str(tmp_path / f"host_program{ext}") for ext in (".hip", ".o", ""))
    with open(src, "w") as f:
        f.write(PRELUDE + main)
    run = lambda cmd, **kw: subprocess.run(cmd, capture_output=True, text=True, **kw)  # noqa: E731
    r = run(["hipcc", "--cuda-host-only", "-O1", "-std=c++17", "-I", ROOT, "-c", src, "-o", obj])
    assert r.returncode == 0, r.stderr
    # without a device pass the kernels' code object is an undefined symbol: nothing loads it
    bundles = set(re.findall(r"__hip_fatbin_[0-9a-f]+", run(["nm", "-u", obj]).stdout))
    r = run(["hipcc", obj, "-o", exe, *[f"-Wl,--defsym={b}=0" for b in bundles]])
    assert r.returncode == 0, r.stderr

    def go(lines):
        r = run([exe], input="\n".join(lines) + "\n", timeout=60)
        assert r.returncode == 0, r.stderr
        return r.stdout.splitlines()
    return go

"""Which kernel a prompt pass's projections take, and what their launcher refuses: host code of the library, asked through a small
program that is compiled here against it (no GPU needed, nothing is launched)."""
import os
import subprocess

import pytest

from paper_2503_08524_amd import build as d3_build

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "d3_common.h"
using namespace d3;

// the launcher's answer to a rotating QKV projection of 4096 columns with one argument that it cannot do with
static int refused(const char* what) {
    static float word;
    static int2 at;
    static float2 cs;
    static int tickets[8];
    GemvArgs a{};
    a.K = 4096; a.total_rows = 3 * 4096; a.ncols = 4096;
    for (int m = 0; m < 3; ++m) a.rows[m] = 4096;
    a.hd = 128; a.H = a.H_kv = 32; a.kv_dtype = 2;
    a.ssq_in = &word; a.ssq_parts = 1; a.col_at = &at; a.rope_cs = &cs; a.part = &word; a.part_tickets = tickets; a.part_bytes = kPromptPartBytes256;
    if (!strcmp(what, "hd")) a.hd = 64;
    if (!strcmp(what, "ssq")) a.ssq_in = nullptr;
    if (!strcmp(what, "col_at")) a.col_at = nullptr;
    if (!strcmp(what, "rope")) a.rope_cs = nullptr;
    if (!strcmp(what, "kv")) a.kv_dtype = 1;
    Tuning tn;
    return launch_gemm_prompt(a, MODE_QKV_ROPE, 256, tn, nullptr, nullptr) == (int)hipErrorInvalidValue;
}

int main(int argc, char** argv) {
    if (argc > 2 && !strcmp(argv[1], "refused")) printf("%d\n", refused(argv[2]));
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if d3_build.is_stale():
        d3_build.build()
    folder = tmp_path_factory.mktemp("choice")
    src, exe = str(folder / "choice.hip"), str(folder / "choice")
    open(src, "w").write(PROGRAM)
    r = subprocess.run([d3_build.HIPCC] + d3_build.FLAGS + ["-I", d3_build.CSRC, "-x", "hip", "--cuda-host-only", "-c", src, "-o", exe + ".o"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([d3_build.HIPCC, exe + ".o", "-o", exe, d3_build.LIB, "-Wl,-rpath," + os.path.dirname(d3_build.LIB)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(*args):
        r = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        return r.stdout.split()
    return run


@pytest.mark.parametrize("what", ["hd", "ssq", "col_at", "rope", "kv"])
def test_rotating_projection_refuses_what_its_epilogue_cannot_do(ask, what):
    # whichever of the two kernels the launch would take
    assert ask("refused", what) == ["1"]

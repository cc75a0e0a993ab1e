"""Which kernel a prompt pass's projections take, and what their launcher refuses: host code of the library, asked through a small
program that is compiled here against it (no GPU needed, nothing is launched)."""
import os
import subprocess

import pytest

from paper_2503_08524_amd import build as d3_build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
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
    if (argc > 5 && !strcmp(argv[1], "large")) printf("%d\n", (int)prompt_takes_large_tiles(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), kPromptPartBytes256, 256, Tuning()));
    if (argc > 1 && !strcmp(argv[1], "tile")) printf("%d\n", tuning_from_env().prompt_tile);
    if (argc > 1 && !strcmp(argv[1], "lines")) {             // d_model, q rows, q + k + v rows, d_ffn, rotating QKV; then any number of columns
        const PromptDims dims{atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6]) != 0};
        Tuning tn;
        for (int i = 7; i < argc; ++i) printf("%d\n", (int)prompt_pass_in_lines(dims, atoi(argv[i]), kPromptPartBytes256, 256, tn));
    }
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


@pytest.mark.parametrize("mode,rows,K,ncols,large", [
    # measured, the smaller tiles / the larger, us: 87 / 99, 90 / 101, 87 / 91, 445 / 458, 142 / 149: few tiles of a short contraction, a last round that leaves compute units idle
    (3, 6144, 2048, 1800, 0), (3, 6144, 2048, 2048, 0), (2, 8192, 2048, 700, 0), (2, 14336, 4096, 1400, 0), (2, 8192, 2048, 1400, 0),
    # 526 / 492, 2482 / 2341, 1334 / 1210, 143 / 134, 397 / 357
    (2, 11008, 4096, 2048, 1), (2, 28672, 8192, 2048, 1), (1, 8192, 28672, 2048, 1), (2, 8192, 3072, 1024, 1), (2, 8192, 2048, 4096, 1)])
def test_estimate_between_the_two_tiles(ask, mode, rows, K, ncols, large):
    assert ask("large", mode, rows, K, ncols) == [str(large)]


@pytest.mark.parametrize("value,tile", [("128", "128"), ("256", "256"), ("129", "0"), ("192", "0"), ("255", "0"), ("64", "0"), ("512", "0")])
def test_tile_override_is_one_of_the_two_or_none(ask, monkeypatch, value, tile):
    monkeypatch.setenv("D3_PROMPT_TILE", value)
    assert ask("tile") == [tile]


WIDTHS = {"7b": (4096, 4096, 12288, 11008, 1), "13b": (5120, 5120, 15360, 13824, 1), "70b": (8192, 8192, 10240, 28672, 1),
          "hd64": (2048, 2048, 3072, 8192, 0), "2048": (2048, 2048, 6144, 8192, 1)}


@pytest.mark.parametrize("width,planes,lines", [("7b", (9, 64, 65, 128, 129, 200, 256, 300), (2048, 4096)), ("13b", (65, 128, 129, 200, 256), (2048, 4096)),
                                                ("70b", (65, 77, 100, 128), (2048, 4096)), ("hd64", (65, 128, 256, 300, 500), (2048, 4096)), ("2048", (128, 256, 300, 512), (4096,))])
def test_form_of_the_split_activations_follows_the_pass(ask, width, planes, lines):
    # rows of lines, 32 k with both halves, are twice as far apart: only where tiles of 256 columns gain more by them (the calls of a few hundred columns are those that lost)
    assert ask("lines", *WIDTHS[width], *planes) == ["0"] * len(planes)
    assert ask("lines", *WIDTHS[width], *lines) == ["1"] * len(lines)

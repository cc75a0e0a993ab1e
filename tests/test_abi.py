"""Host-side checks of the C ABI (no GPU): the library loads, exports every symbol the header
declares, and the host-only schedule entry point agrees with the oracle bit for bit."""
import os
import re

import numpy as np
import pytest

import d3_inputs
import paper_2503_08524_amd as d3
from oracle import oracle
from paper_2503_08524_amd import build as d3_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if d3_build.is_stale():
        d3_build.build()
    return d3.load_library()


def declared_functions():
    text = open(os.path.join(ROOT, "include", "d3.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(d3_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol(lib):
    names = declared_functions()
    assert {"d3_plan_depth", "d3_prefill", "d3_decode_step", "d3_fill_missing_kv", "d3_create", "d3_destroy",
            "d3_set_plan", "d3_workspace_size", "d3_last_error", "d3_n_ctx"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n


@pytest.mark.parametrize("L,alpha,start", [(4, 0.97, 2), (32, 0.995, 19), (32, 0.99, 19), (40, 0.995, 24), (80, 0.995, 48),
                                           (32, 1.0, 19), (32, 0.8, 0), (80, 0.9999, 16), (40, 0.9, 39)])
def test_plan_is_bit_exact_against_oracle(lib, L, alpha, start):
    for min_keep in (0, 2):
        got = d3.d3_plan_depth(L, alpha, start, min_keep, 1300)
        ref = oracle.plan_depth(L, alpha, start, min_keep, 1300)
        for g, r in zip(got, ref):
            assert (g == r).all()


@pytest.mark.parametrize("L,first,last,start", [(32, 32, 8, 0), (32, 32, 17, 31), (40, 36, 4, 24), (80, 80, 0, 48), (4, 4, 1, 2), (32, 20, 20, 5)])
def test_linear_plan_is_bit_exact_against_oracle_and_survives_the_table_entry(lib, L, first, last, start):
    for n in (1, 2, 77, 1024):
        got = d3.d3_plan_depth_linear(L, first, last, start, n)
        ref = oracle.plan_depth_linear(L, first, last, start, n)
        for g, r in zip(got, ref):
            assert (g == r).all()
        assert (d3.d3_plan_from_table(L, ref[0], ref[1]) == ref[2]).all()


def test_plan_table_rejects_steps_that_do_not_fit(lib):
    for keep, drop in [([5], [0]), ([-1], [0]), ([2], [3]), ([2], [-1]), ([4, 3, 1], [0, 0, 2])]:
        with pytest.raises(d3.D3Error) as e:
            d3.d3_plan_from_table(4, keep, drop)
        assert e.value.status == -1 and "d3_plan_from_table" in str(e.value)
    assert d3.d3_plan_from_table(4, [4, 3, 0], [4, 3, 0]).tolist() == [[0, 1, 2, 3], [0, 1, 2, -1], [-1, -1, -1, -1]]
    with pytest.raises(d3.D3Error):
        d3.d3_plan_depth_linear(8, 9, 2, 0, 4)


def test_plan_from_table_lists_exactly_the_blocks_outside_each_window(lib):
    rng = np.random.default_rng(7)
    for _ in range(200):
        L = int(rng.integers(1, 90))
        n = int(rng.integers(1, 40))
        keep = rng.integers(0, L + 1, size=n)
        drop = np.array([int(rng.integers(0, k + 1)) for k in keep])       # window [drop, drop + L - keep) ends at or before L
        ids = d3.d3_plan_from_table(L, keep, drop)
        for i in range(n):
            want = [l for l in range(L) if not (drop[i] <= l < drop[i] + L - keep[i])]
            assert ids[i, : keep[i]].tolist() == want and (ids[i, keep[i]:] == -1).all()


def test_plan_accepts_null_outputs_and_zero_steps(lib):
    assert lib.d3_plan_depth(8, 0.9, 3, 0, 5, None, None, None) == 0
    assert lib.d3_plan_depth(8, 0.9, 3, 0, 0, None, None, None) == 0


@pytest.mark.parametrize("args", [(0, 0.9, 0, 0, 4), (4, 0.0, 0, 0, 4), (4, 1.0001, 0, 0, 4), (4, float("nan"), 0, 0, 4),
                                  (4, 0.9, 4, 0, 4), (4, 0.9, -1, 0, 4), (4, 0.9, 0, 5, 4), (4, 0.9, 0, -1, 4), (4, 0.9, 0, 0, -1)])
def test_plan_rejects_bad_arguments(lib, args):
    with pytest.raises(d3.D3Error) as e:
        d3.d3_plan_depth(*args)
    assert e.value.status == -1 and "d3_plan_depth" in str(e.value)


def test_workspace_size_and_shape_checks(lib):
    for s in (d3_inputs.TINY, d3_inputs.LLAMA_7B, d3_inputs.LLAMA_13B, d3_inputs.LLAMA_70B):
        n = d3.d3_workspace_size(s, "f16" if s.dtype == "bf16" else "f32", 8, 2048)
        assert n > 0 and n % 256 == 0 and n < 2 ** 31
    bad = d3_inputs.ModelShape("bad", L=2, d=256, H=4, H_kv=3, hd=64, F=688, V=1024)
    assert d3.d3_workspace_size(bad, "f16", 1, 64) == 0
    assert "n_kv_heads" in lib.d3_last_error().decode()
    bad = d3_inputs.ModelShape("bad", L=2, d=256, H=4, H_kv=4, hd=80, F=688, V=1024)
    assert d3.d3_workspace_size(bad, "f16", 1, 64) == 0
    assert d3.d3_workspace_size(d3_inputs.TINY, "f32", 33, 64) == 0          # max_batch beyond 32
    assert d3.d3_workspace_size(d3_inputs.LLAMA_7B, "bf16", 1, 64) == 0       # a bf16 cache misses the logit tolerance
    assert "D3_BF16" in lib.d3_last_error().decode()


def test_workspace_of_an_fp32_cache_is_that_of_passes_of_2048_columns(lib):
    # wider passes pay with tiles of 256 columns, which an fp32 cache does not take
    for s in (d3_inputs.LLAMA_7B, d3_inputs.LLAMA_70B):
        assert d3.d3_workspace_size(s, "f32", 1, 2048) == d3.d3_workspace_size(s, "f32", 1, 4096) == d3.d3_workspace_size(s, "f32", 8, 4096)
        assert d3.d3_workspace_size(s, "f16", 1, 2048) < d3.d3_workspace_size(s, "f16", 1, 4096)


SMALLER = [  # (shape, cache, max_batch, max_seq, bytes that d3_workspace_size gave when passes were at most 2048 columns and those of the vector ALUs of one sequence)
    (d3_inputs.TINY, "f32", 8, 512, 8929792), (d3_inputs.TINY, "f32", 32, 128, 3172864),
    (d3_inputs.LLAMA_7B, "f16", 1, 64, 115599104), (d3_inputs.LLAMA_7B, "f16", 1, 300, 168193792), (d3_inputs.LLAMA_7B, "f16", 8, 512, 510059264),
    (d3_inputs.LLAMA_13B, "f16", 32, 2048, 619504384), (d3_inputs.LLAMA_70B, "f32", 8, 2048, 935256832), (d3_inputs.LLAMA_70B, "f16", 8, 2048, 935256832),
    (d3_inputs.ModelShape("f32", L=2, d=2048, H=16, H_kv=16, hd=128, F=5504, V=32000, dtype="f32"), "f32", 32, 128, 26198784),
    (d3_inputs.ModelShape("hd64", L=3, d=2048, H=32, H_kv=8, hd=64, F=8192, V=32000, dtype="bf16"), "f16", 1, 300, 123527680),
    (d3_inputs.ModelShape("odd", L=3, d=264, H=4, H_kv=2, hd=64, F=696, V=1000, dtype="bf16"), "f16", 32, 128, 3060224),
    # few MLP rows, and passes whose columns are no multiple of 256
    (d3_inputs.ModelShape("narrow-mlp", L=1, d=1536, H=12, H_kv=12, hd=128, F=128, V=512, dtype="bf16"), "f16", 1, 320, 81393408),
    (d3_inputs.ModelShape("wide", L=1, d=8192, H=16, H_kv=8, hd=128, F=1088, V=32000, dtype="bf16"), "f32", 2, 146, 133369600),
    (d3_inputs.ModelShape("hd64-narrow", L=1, d=2048, H=16, H_kv=2, hd=64, F=128, V=32000, dtype="bf16"), "f32", 16, 1658, 137675264)]


@pytest.mark.parametrize("shape,kv,B,n,size", SMALLER)
def test_smaller_workspaces_are_accepted(lib, shape, kv, B, n, size):
    """The sizes above, with which contexts used to be made, are enough still; a tenth is refused.  Without a GPU d3_create stops at the device, behind the workspace's check."""
    import ctypes as C
    import torch
    from paper_2503_08524_amd import binding
    if torch.cuda.is_available():
        pytest.skip("the buffers below are not the GPU's")
    word = np.zeros(1024, np.uint8)
    at = (word.ctypes.data + 255) // 256 * 256
    layers = (binding._LayerWeights * shape.L)(*[binding._LayerWeights(*[at] * 9) for _ in range(shape.L)])
    desc, w, ctx = binding._desc(shape, kv, B, n), binding._Weights(at, layers, at, at), C.c_void_p()

    def create(bytes_):
        return lib.d3_create(C.byref(ctx), C.byref(desc), C.byref(w), at, at, at, bytes_), lib.d3_last_error().decode()
    device = create(binding.d3_workspace_size(shape, kv, B, n))[0]
    status, message = create(size)
    assert status == device, message
    status, message = create(size // 10)
    assert status == -1 and "workspace" in message and status != device


def test_workspace_of_the_vector_alus_holds_no_split_activations(lib):
    # x, q k v, attention, MLP and rotary rows of 4096 / 2 columns and little else: the bf16 halves and sums of squares belong to the matrix cores, whose MLP rows are 32
    d, F, C = 4096, 11008, 2048
    f32 = d3_inputs.ModelShape("f32", L=2, d=d, H=32, H_kv=32, hd=128, F=F, V=32000, dtype="f32")
    small = 32 * 32 * 32 * 130 * 4 + 32 * (32000 + d) * 4 + C * (32 * 4 + 64 * 8) + (1 << 16)
    assert C * 4 * (d + 3 * d + d + F) < d3.d3_workspace_size(f32, "f32", 32, 128) < C * 4 * (d + 3 * d + d + F) + small
    parts, split = 64 << 20, C * 4 * (d + F + d)
    assert d3.d3_workspace_size(d3_inputs.LLAMA_7B, "f32", 32, 128) < C * 4 * (5 * d) + split + parts + small + C * (2048 + 8) + 32 * (F + d) * 4


def test_workspace_holds_partial_sums_only_where_a_kernel_can_write_them(lib):
    MiB = 1 << 20
    shape = d3_inputs.ModelShape("small", L=2, d=256, H=4, H_kv=4, hd=64, F=704, V=1024, dtype="bf16")
    # fp32 models never run K-sliced: 32 columns of activations, attention partials and logits are a few MiB
    assert d3.d3_workspace_size(d3_inputs.TINY, "f32", 4, 128) < 12 * MiB
    # a small bf16 model in one column block: the panel kernel's 16 MiB; 6 row blocks in 8 parts of 128 KiB would be 6
    small = d3.d3_workspace_size(shape, "f16", 1, 128)
    assert 16 * MiB < small < 16 * MiB + 12 * MiB
    # in sixteen column blocks: 6 x 16 tiles in 8 parts are more than a launch may publish, 64 MiB
    long = d3.d3_workspace_size(shape, "f16", 1, 2048)
    activations = lambda C: C * (4 * (256 + 768 + 256) + 2 * 2 * (256 + 704 + 256) + 8 * 32 + 4 * 512 + 4 * 4)
    assert abs((long - small) - (48 * MiB + activations(2048) - activations(128))) < MiB
    # 7B widths, 48 QKV and 86 gate/up row blocks: one column block can already publish 64 MiB (86 x 8 parts)
    assert d3.d3_workspace_size(d3_inputs.LLAMA_7B, "f16", 1, 64) > 64 * MiB


def test_null_context_is_an_error_not_a_crash(lib):
    assert lib.d3_set_plan(None, 0.9, 0, 0, 4) == -1
    assert lib.d3_decode_step(None, None, 1, None, None, None, None) == -1
    assert lib.d3_prefill(None, None, 1, 1, 0, None, None, None, None) == -1
    assert lib.d3_fill_missing_kv(None, 0, 0, 0, None) == -1
    assert lib.d3_n_ctx(None) == 0
    assert lib.d3_destroy(None) == 0

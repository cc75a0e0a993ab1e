"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same
seeded inputs, element by element.  Bars: schedule bit-exact (tests/test_abi.py), logits within
2e-2 max abs, hidden state within 1e-2 relative L2 after every executed block, greedy tokens
identical on the small configurations."""
import numpy as np
import pytest

import d3_inputs
from d3_inputs import ModelShape
from tests import helpers

pytestmark = pytest.mark.gpu

# small shapes that still span several tiles and ragged tails of every kernel
SMALL_BF16 = ModelShape("small-bf16", L=4, d=256, H=4, H_kv=4, hd=64, F=704, V=1024, dtype="bf16")
SMALL_GQA = ModelShape("small-gqa", L=3, d=512, H=8, H_kv=2, hd=128, F=1376, V=2000, dtype="bf16")


def _forced(B, G, V, seed):
    return d3_inputs.make_prompt(B, max(G - 1, 1), V, seed=seed)


def _run(shape, B, P, G, alpha, start, kv_dtype=None, forced_seed=None, check_tokens="margin", seed=0, **kw):
    w = d3_inputs.make_weights(shape, seed)
    prompts = d3_inputs.make_prompt(B, P, shape.V, seed=1)
    forced = None if forced_seed is None else _forced(B, G, shape.V, forced_seed)
    print(f"case {shape.name} B={B} P={P} G={G} alpha={alpha} start={start} kv={kv_dtype}", flush=True)
    gpu = helpers.gpu_generate(shape, w, prompts, G, alpha, start, forced=forced, kv_dtype=kv_dtype, **kw)
    _, gens = helpers.oracle_generate(shape, w, prompts, G, alpha, start, forced=forced, min_keep=kw.get("min_keep", 0),
                                      linear=kw.get("linear"), lengths=kw.get("lengths"))
    wl, wh = helpers.compare(gpu, gens, G, check_tokens=check_tokens)
    print(f"  worst logit abs err {wl:.3e}, worst hidden rel L2 {wh:.3e}", flush=True)
    return gpu, gens


@pytest.mark.parametrize("alpha", [0.97, 1.0])
def test_tiny_config_tokens_logits_hidden(alpha):
    # the first benchmark configuration in full: fp32 weights, fp32 cache, free-running greedy decoding
    gpu, gens = _run(d3_inputs.TINY, 1, 16, 32, alpha, 2, kv_dtype="f32", check_tokens="all")
    helpers.compare(gpu, gens, 32, check_tokens="all", logit_atol=1e-4, hidden_tol=1e-5)


@pytest.mark.parametrize("start", [0, 2, 3])
def test_tiny_config_linear_decay_shallow_middle_and_deep_first(start):
    # the comparison schedules (linear decay; windows that grow from the first block, the middle, the last block)
    # are plans for the same kernels: free-running greedy decoding, tokens identical
    gpu, gens = _run(d3_inputs.TINY, 1, 16, 32, 1.0, start, kv_dtype="f32", check_tokens="all", linear=(4, 1))
    helpers.compare(gpu, gens, 32, check_tokens="all", logit_atol=1e-4, hidden_tol=1e-5)
    assert [h.shape[0] - 1 for h in gpu["hidden"][1:]] == gens[0].keep[1:32].tolist()


def test_batched_linear_decay_on_the_matrix_cores():
    gpu, gens = _run(SMALL_GQA, 5, 21, 12, 1.0, 0, forced_seed=3, linear=(3, 1))
    gpu, gens = _run(SMALL_BF16, 17, 9, 10, 1.0, 3, forced_seed=4, linear=(4, 0))


@pytest.mark.parametrize("shape,lengths,kv", [
    (d3_inputs.TINY, (16, 5, 11), "f32"),                 # fp32 weights: vector-ALU projections, one column per launch group
    (SMALL_BF16, (9, 70, 1, 33, 64), None),               # head_dim 64: vector-ALU attention; one sequence a pass
    (SMALL_GQA, (130, 17, 77, 130), "f16"),               # head_dim 128, f16 cache: one pass for all of them, MFMA attention in decode
    (SMALL_GQA, (40, 3), "f32"),
])
def test_left_padded_batch_of_unequal_prompts(shape, lengths, kv):
    # every sequence of a ragged batch must behave as if it had run alone: its own positions, its own context
    B, P = len(lengths), max(lengths)
    _run(shape, B, P, 9, 0.8, 1, kv_dtype=kv, forced_seed=21, lengths=np.array(lengths, np.int32), max_seq=P + 9)


@pytest.mark.parametrize("lengths,kv", [((130, 17, 77), "f16"), ((40, 300, 1), "f32")])
def test_left_padded_batch_one_sequence_a_pass(monkeypatch, lengths, kv):
    # without the panel and LDS-tiled kernels a pass is 32 columns of one sequence: query tiles whose rows begin above row 0
    monkeypatch.setenv("D3_MFMA_WIDE", "0")
    gpu, gens = _run(SMALL_GQA, len(lengths), max(lengths), 3, 0.8, 1, kv_dtype=kv, forced_seed=21, lengths=np.array(lengths, np.int32), max_seq=max(lengths) + 3)
    if kv == "f32":     # only arithmetic rounding is left
        helpers.compare(gpu, gens, 3, logit_atol=2e-4, hidden_tol=1e-4)


def test_left_padded_batch_spans_attention_splits():
    # the short sequence's rows begin inside a later split: the splits below it hold nothing of it
    lengths = np.array([700, 150, 699], np.int32)
    _run(SMALL_GQA, 3, 700, 6, 0.7, 1, forced_seed=22, lengths=lengths)
    _run(SMALL_BF16, 2, 650, 4, 0.9, 2, forced_seed=23, lengths=np.array([40, 650], np.int32))


def test_bf16_shape_that_does_not_fit_the_matrix_core_tiles():
    # d_model, d_ffn not multiples of 32, vocab not a multiple of 16: batched passes stay on the vector-ALU projections
    shape = ModelShape("odd-bf16", L=3, d=264, H=4, H_kv=2, hd=64, F=696, V=1000, dtype="bf16")
    _run(shape, 3, 21, 7, 0.8, 1, forced_seed=31)
    _run(shape, 5, 40, 5, 0.8, 0, forced_seed=32, lengths=np.array([40, 7, 33, 1, 40], np.int32))


def test_tiny_config_f16_cache():
    _run(d3_inputs.TINY, 1, 16, 32, 0.97, 2, kv_dtype="f16", forced_seed=5)


def test_bf16_cache_is_refused():
    # its 8-bit mantissa puts the logits outside the tolerance after two blocks at real widths
    from paper_2503_08524_amd import binding
    w = binding.weights_to_device(SMALL_BF16, d3_inputs.make_weights(SMALL_BF16, 0))
    with pytest.raises(binding.D3Error) as e:
        binding.Decoder(SMALL_BF16, w, 1, 32, kv_dtype="bf16")
    assert "D3_BF16" in str(e.value)


@pytest.mark.parametrize("B", [1, 2, 3, 4])
def test_tiny_fp32_batches_use_the_alu_path(B):
    _run(d3_inputs.TINY, B, 9, 8, 0.9, 1, kv_dtype="f32", forced_seed=6)


# Groups of columns in one launch of the vector-ALU projections: 4, 2 and 1 columns a workgroup (rows of up to 15 KB, 30 KB and 60 KB of fp32 activations), batches that fill their
# last group and that do not, group by group in decode and in prompt passes of several sequences (15 to 350 columns in one pass, beside a ragged batch, which stays
# one sequence a pass), fp32 and bf16 rows (bf16: widths that the matrix cores do not take), a cache of 16 bits
@pytest.mark.parametrize("B,P,d,F,dtype,kv,lengths", [
    (5, 3, 256, 688, "f32", "f32", None), (8, 40, 256, 688, "f32", "f32", None), (9, 33, 256, 688, "f32", "f16", None), (32, 5, 256, 688, "f32", "f32", None), (3, 97, 256, 688, "f32", "f32", None),
    (5, 7, 256, 6000, "f32", "f32", None), (3, 20, 256, 12000, "f32", "f32", None), (7, 50, 264, 696, "bf16", "f32", None), (3, 70, 256, 688, "f32", "f32", (70, 1, 41))])
def test_groups_of_columns_on_the_vector_alus(B, P, d, F, dtype, kv, lengths):
    s = ModelShape("groups", L=2, d=d, H=4, H_kv=2, hd=64, F=F, V=1000, dtype=dtype)
    kw = {} if lengths is None else {"lengths": np.array(lengths, np.int32)}
    gpu, gens = _run(s, B, P, 3, 0.8, 1, kv_dtype=kv, forced_seed=6, **kw)
    if kv == "f32":
        helpers.compare(gpu, gens, 3, logit_atol=1e-4, hidden_tol=1e-5)


ODD_BF16 = ModelShape("odd-bf16", L=2, d=264, H=4, H_kv=2, hd=64, F=696, V=1000, dtype="bf16")


# prompts in more than one pass: 40 positions of 5 sequences in passes of 12, 12, 12 and 4 (64 columns, which 5 does not divide), 130 of one in three, 70 of a ragged batch in
# passes of 64 and 6; 1200 columns of 3 sequences, whose contexts are cut from 128 rows on, in the passes that the partials leave
@pytest.mark.parametrize("shape,B,P,cols,lengths", [(d3_inputs.TINY, 5, 40, 64, None), (ODD_BF16, 5, 40, 64, None), (d3_inputs.TINY, 1, 130, 64, None), (ODD_BF16, 3, 70, 64, (70, 1, 41)),
                                                    (d3_inputs.TINY, 3, 400, 0, None), (ODD_BF16, 1, 1100, 0, None)])
def test_prompts_of_several_passes_on_the_vector_alus(monkeypatch, shape, B, P, cols, lengths):
    if cols:
        monkeypatch.setenv("D3_PREFILL_COLS", str(cols))
    kw = {} if lengths is None else {"lengths": np.array(lengths, np.int32)}
    gpu, gens = _run(shape, B, P, 3, 0.8, 1, kv_dtype="f32", forced_seed=6, **kw)
    helpers.compare(gpu, gens, 3, logit_atol=1e-4, hidden_tol=1e-5)


NARROW_MLP = ModelShape("narrow-mlp", L=1, d=1536, H=12, H_kv=12, hd=128, F=128, V=512, dtype="bf16")


@pytest.mark.parametrize("shape,kv,B,P,size,tile", [
    (ModelShape("smaller-ws", L=1, d=1536, H=12, H_kv=12, hd=128, F=2048, V=512, dtype="bf16"), "f16", 2, 590, 153336576, None),      # the smaller part buffer, 1280 columns
    (d3_inputs.TINY, "f32", 8, 505, 8929792, None), (d3_inputs.TINY, "f32", 32, 120, 3172864, None),       # passes of one sequence's columns, of all of them
    (NARROW_MLP, "f16", 1, 310, 81393408, None), (NARROW_MLP, "f16", 1, 310, 81393408, "256")])            # split activations of 384 columns, which tiles of 256 would read 512 of
def test_prompts_in_a_workspace_of_an_earlier_size(monkeypatch, shape, kv, B, P, size, tile):
    # max_seq 600, 512, 128 and 320: what d3_workspace_size gave for them when it asked for less
    import torch
    from paper_2503_08524_amd import binding
    w, toks = binding.weights_to_device(shape, d3_inputs.make_weights(shape, 0), "cuda:0"), torch.from_numpy(d3_inputs.make_prompt(B, P, shape.V, seed=1)).to("cuda:0")
    rows = {590: 600, 505: 512, 120: 128, 310: 320}[P]
    if tile:
        monkeypatch.setenv("D3_PROMPT_TILE", tile)
    print(f"case smaller workspace {shape.name} B={B} P={P}", flush=True)

    def run():
        dec, logits = binding.Decoder(shape, w, B, rows, kv_dtype=kv), torch.zeros(B, shape.V, device="cuda:0")
        dec.prefill(toks, logits=logits)
        torch.cuda.synchronize()
        got = logits.double(), dec.k_cache.double(), dec.v_cache.double(), dec.workspace.numel()
        dec.close()
        return got
    full = run()
    monkeypatch.setattr(binding.load_library(), "d3_workspace_size", lambda desc: size)
    less = run()
    assert less[3] == size < full[3]
    # another cut of the passes moves sums by their rounding: an ulp of an fp16 row (4.9e-4, and a row in a hundred), a few of fp32
    for a, b in zip(less[:3], full[:3]):
        assert (a - b).norm() / b.norm() < (1e-3 if kv == "f16" else 2e-6)


@pytest.mark.parametrize("B,P,past", [(1, 700, 0), (3, 1100, 0), (8, 300, 0), (5, 70, 1500), (2, 1032, 40)])
def test_contexts_of_vector_alu_prompts_are_cut_as_passes_of_32_columns_cut_them(monkeypatch, B, P, past):
    # long contexts: logits and cache rows of a batch in wide passes, bit for bit those in passes of 64 columns and those of each sequence alone
    import torch
    from paper_2503_08524_amd import binding
    s = d3_inputs.TINY
    w = binding.weights_to_device(s, d3_inputs.make_weights(s, 3), "cuda:0")
    toks = torch.from_numpy(d3_inputs.make_prompt(B, past + P, s.V, seed=4)).to("cuda:0")
    print(f"case cut contexts B={B} P={P} past={past}", flush=True)

    def run(t):
        dec, lg = binding.Decoder(s, w, t.shape[0], past + P, kv_dtype="f32"), torch.zeros(t.shape[0], s.V, device="cuda:0")
        if past:
            dec.prefill(t[:, :past].contiguous())
        dec.prefill(t[:, past:].contiguous(), pos_begin=past, logits=lg)
        torch.cuda.synchronize()
        got = lg, dec.k_cache.clone(), dec.v_cache.clone()
        dec.close()
        return got
    lg, k, v = run(toks)
    for b in range(B):
        one = run(toks[b:b + 1].contiguous())
        assert torch.equal(one[0][0], lg[b]) and torch.equal(one[1][:, 0], k[:, b]) and torch.equal(one[2][:, 0], v[:, b])
    monkeypatch.setenv("D3_PREFILL_COLS", "64")
    assert all(torch.equal(a, b) for a, b in zip(run(toks), (lg, k, v)))


def test_batch_on_the_vector_alus_equals_its_sequences_one_at_a_time():
    # the sums of a column do not depend on the group it is in: logits and cache rows of a batch, prompt and decode step, bit for bit those of each sequence alone
    # (16 rows: attention cuts neither context)
    import torch
    from paper_2503_08524_amd import binding
    s = d3_inputs.TINY
    w, B, P = binding.weights_to_device(s, d3_inputs.make_weights(s, 3), "cuda:0"), 7, 16
    toks = torch.from_numpy(d3_inputs.make_prompt(B, P, s.V, seed=4)).to("cuda:0")
    print("case batch against its sequences", flush=True)

    def run(t):
        n = t.shape[0]
        dec = binding.Decoder(s, w, n, P + 2, kv_dtype="f32")
        out, lg = torch.zeros(n, dtype=torch.int32, device="cuda:0"), torch.zeros(2, n, s.V, device="cuda:0")
        dec.prefill(t, next_tok=out, logits=lg[0])
        dec.set_plan_table([s.L, s.L], [0, 0])
        dec.decode_step(t[:, 0].contiguous(), 1, out, logits=lg[1])
        torch.cuda.synchronize()
        got = lg.clone(), dec.k_cache.clone(), dec.v_cache.clone()
        dec.close()
        return got
    lg, k, v = run(toks)
    for b in range(B):
        one = run(toks[b:b + 1].contiguous())
        assert torch.equal(one[0][:, 0], lg[:, b]) and torch.equal(one[1][:, 0, :, :P + 1], k[:, b, :, :P + 1]) and torch.equal(one[2][:, 0, :, :P + 1], v[:, b, :, :P + 1])


@pytest.mark.parametrize("B,P", [(1, 16), (2, 7), (5, 13), (16, 3), (17, 4), (32, 2)])
def test_small_bf16_matrix_core_path(B, P):
    # B = 1 decodes on the vector ALUs and prefills on the matrix cores; B >= 2 uses the matrix cores throughout
    _run(SMALL_BF16, B, P, 8, 0.9, 2, forced_seed=7)


# split activations in planes: decode and prompt passes of 9 to 16 columns, heads of as many and of fewer columns behind them, heads of 9 to 16 columns behind a wider
# pass, contractions whose last turn is ragged, grouped queries
@pytest.mark.parametrize("B,P,d,F,H_kv,kv", [(9, 1, 96, 160, 2, "f32"), (16, 1, 256, 416, 1, "f16"), (1, 13, 96, 160, 1, "f32"), (3, 4, 160, 96, 2, "f32"), (8, 2, 256, 224, 2, "f32"),
                                             (12, 3, 160, 288, 1, "f32"), (16, 9, 256, 512, 2, "f32"), (1, 75, 96, 160, 2, "f32"), (11, 5, 32, 32, 1, "f16")])
def test_nine_to_sixteen_columns(B, P, d, F, H_kv, kv):
    s = ModelShape("planes", L=3, d=d, H=2, H_kv=H_kv, hd=64, F=F, V=512, dtype="bf16")
    gpu, gens = _run(s, B, P, 4, 0.97, 2, forced_seed=19, kv_dtype=kv)
    helpers.compare(gpu, gens, 4, **({} if kv == "f16" else {"logit_atol": 2e-4, "hidden_tol": 1e-4}))


@pytest.mark.parametrize("shape,B,P", [(SMALL_BF16, 2, 24), (SMALL_BF16, 2, 97), (SMALL_BF16, 1, 81), (SMALL_GQA, 1, 80),
                                       (SMALL_GQA, 2, 72), (SMALL_GQA, 1, 128), (SMALL_BF16, 2, 50), (SMALL_GQA, 1, 168),
                                       (SMALL_GQA, 1, 136), (SMALL_BF16, 1, 144), (SMALL_GQA, 2, 145), (SMALL_GQA, 1, 72), (SMALL_GQA, 1, 145),
                                       (SMALL_GQA, 1, 7), (SMALL_GQA, 1, 13)])
def test_prompt_lengths_that_end_in_every_chunk_width(shape, B, P):
    # a pass is one sequence at batch 1 and at head_dim 64, both sequences end to end at batch 2 and head_dim 128: passes of 24, 97,
    # 81, 80, 72, 128, 50, 168, 136, 144, 145, 7 and 13 columns, and of 144 and 290 shared ones.  They end in each of the projection
    # kernels (packed, 16-column, the panel kernel with two, four and eight column tiles, and the LDS-tiled kernel with a ragged second
    # or third column block) and of the attention paths of a prompt pass (per column on the vector ALUs at head_dim 64; at 128 query tiles for one
    # sequence of so few columns, the whole-context kernel for several)
    _run(shape, B, P, 4, 0.8, 1, forced_seed=9)


def test_wide_prompt_chunks_as_two_launches_of_64_columns(monkeypatch):
    # what the panel kernel does with a pass of more than 64 columns on large matrices (hundreds of MB), forced on small ones: 100 columns of
    # one sequence, 2 x 50 shared ones, 97 at head_dim 64; 2 x 150 columns are the LDS-tiled kernel's, whatever the matrix
    monkeypatch.setenv("D3_WIDE_SPLIT_MB", "0")
    _run(SMALL_GQA, 1, 100, 4, 0.8, 1, forced_seed=9)
    _run(SMALL_GQA, 2, 50, 4, 0.8, 1, forced_seed=9)
    _run(SMALL_GQA, 2, 150, 4, 0.8, 1, forced_seed=9)
    _run(SMALL_BF16, 1, 97, 4, 0.8, 1, forced_seed=9)


@pytest.mark.parametrize("B", [1, 2])
@pytest.mark.parametrize("cols", [64, 128, 256])
def test_prompt_chunks_of_a_forced_width(monkeypatch, cols, B):
    # prompts in passes of 64 or 128 columns (panel kernel) and of 256 (LDS-tiled kernel).  One sequence: 150 tokens in 64 + 64 + 22, 700 in
    # five passes of 128 and one of 60, or two of 256 and one of 188 (second column block ragged); all but the first begin above row 0.
    # Two sequences end to end: 300 columns in four passes of 64 and one of 44, 1400 in ten of 128 and one of 120, or five of 256 and one of 120
    monkeypatch.setenv("D3_PREFILL_COLS", str(cols))
    _run(SMALL_GQA, B, 150 if cols == 64 else 700, 4, 0.8, 1, forced_seed=9)


@pytest.mark.parametrize("wgs", [1, 1 << 20])
@pytest.mark.parametrize("B,P,cols", [(1, 300, 128), (1, 470, 256), (2, 300, 128)])
@pytest.mark.parametrize("kv", ["f16", "f32"])
def test_prompt_of_several_passes_on_either_attention_kernel(monkeypatch, kv, B, P, cols, wgs):
    # passes whose first position lies above row 0, on the whole-context kernel (wgs 1) and on query tiles: one sequence a pass, and two
    # that share passes
    monkeypatch.setenv("D3_PROMPT_ATTN_WGS", str(wgs))
    monkeypatch.setenv("D3_PREFILL_COLS", str(cols))
    gpu, gens = _run(SMALL_GQA, B, P, 2, 0.8, 1, forced_seed=9, kv_dtype=kv)
    if kv == "f32":     # only arithmetic rounding is left
        helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("B,P,cols,lengths,kv", [(2, 32, 64, None, "f16"), (5, 13, 64, None, "f32"), (3, 43, 128, None, "f16"), (3, 150, 256, None, "f16"),
                                                (32, 7, 0, None, "f32"), (4, 90, 128, (90, 1, 37, 2), "f32"), (3, 260, 320, (64, 260, 65), "f16")])
def test_sequences_share_prompt_passes(monkeypatch, B, P, cols, lengths, kv):
    # prompts laid end to end and cut into passes: passes that end between sequences, inside one and one column into the next (65 = 64
    # + 1 and 129 = 128 + 1 columns: a pass of a single column), runs of one column, 32 sequences in a pass, and unequal prompts padded on the left; hidden states of the
    # last positions from every pass, logits from the one head at the end
    if cols:
        monkeypatch.setenv("D3_PREFILL_COLS", str(cols))
    s = ModelShape("shared", L=2, d=256, H=4, H_kv=2, hd=128, F=384, V=512, dtype="bf16")
    gpu, gens = _run(s, B, P, 2, 1.0, 1, forced_seed=19, kv_dtype=kv, lengths=None if lengths is None else np.array(lengths, np.int32), max_seq=P + 2)
    if kv == "f32":     # only arithmetic rounding is left
        helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("B,P,cols,lengths,alone", [(3, 1, 0, None, (0, 1, 2)), (7, 1, 0, None, range(7)), (2, 65, 64, None, (0, 1)), (2, 129, 64, None, (0, 1)),
                                                     (4, 90, 128, (90, 1, 37, 1), (1, 3)), (3, 65, 64, (65, 64, 1), (0, 2))])
def test_last_columns_that_stand_alone_keep_the_fp32_projections(monkeypatch, B, P, cols, lengths, alone):
    # a prompt of one token, or of whole chunks and one, ends in a pass of a single column on the fp32 projections; in a batch
    # it must not join the shared pass of bf16 hi + lo activations (2^-17 per activation).  What that column computes itself stays in
    # fp32: sums of up to 384 products of 24 bits, rounded at most 2^-24 x sqrt(384) = 1.2e-6 off; with a prompt before it, block 0
    # (slot 1) also sees cache rows of the shared passes through softmax weights that sum to one.
    if cols:
        monkeypatch.setenv("D3_PREFILL_COLS", str(cols))
    s = ModelShape("alone", L=2, d=256, H=4, H_kv=2, hd=128, F=384, V=512, dtype="bf16")
    gpu, gens = _run(s, B, P, 2, 1.0, 1, forced_seed=19, kv_dtype="f32", lengths=None if lengths is None else np.array(lengths, np.int32), max_seq=P + 2)
    for b in range(B):
        hr, hg = gens[b].hidden[0], gpu["hidden"][0][:, b].astype(np.float64)
        rel = np.linalg.norm(hg - hr, axis=1) / np.linalg.norm(hr, axis=1)
        lg = np.abs(gpu["logits"][0][b] - gens[b].logits[0]).max() / np.abs(gens[b].logits[0]).max()
        print(f"  seq {b} {'alone' if b in alone else 'shared'} hidden {rel} logits {lg:.2e}", flush=True)
        if b in alone:
            assert rel.max() <= 1.2e-6 and lg <= 1.2e-6, f"seq {b}"


@pytest.mark.parametrize("B,P,wgs", [(3, 150, 1), (2, 700, 1 << 20), (5, 1, 0)])
def test_prompt_pass_of_a_batch_replays_from_a_graph(monkeypatch, B, P, wgs):
    # shared passes on the whole-context kernel and on query tiles run by run (arrival counters of splits and K parts must be left
    # zero by every replay), and lone tokens on the fp32 projections: each replay equals the eager call, bit for bit
    import torch
    from paper_2503_08524_amd import binding
    if wgs:
        monkeypatch.setenv("D3_PROMPT_ATTN_WGS", str(wgs))
    monkeypatch.setenv("D3_PROMPT_KS", "2")
    s = ModelShape("graph", L=2, d=256, H=4, H_kv=2, hd=128, F=704, V=512, dtype="bf16")
    dec = binding.Decoder(s, binding.random_weights_on_device(s, 5), B, P + 2)
    toks = [torch.from_numpy(d3_inputs.make_prompt(B, P, s.V, seed=k)).to("cuda:0") for k in (1, 2)]
    fed, out, logits = toks[0].clone(), torch.zeros(B, dtype=torch.int32, device="cuda:0"), torch.zeros(B, s.V, device="cuda:0")
    print(f"case graph B={B} P={P} wgs={wgs}", flush=True)
    want = []
    for t in toks:
        dec.prefill(t, next_tok=out, logits=logits)
        want.append((out.clone(), logits.clone(), dec.k_cache.clone()))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dec.prefill(fed, next_tok=out, logits=logits)
    for k in (0, 1, 1, 0, 1):
        fed.copy_(toks[k])
        logits.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[k][0]) and torch.equal(logits, want[k][1]) and torch.equal(dec.k_cache, want[k][2])
    dec.close()


def test_hidden_states_of_shared_passes_into_a_buffer_aligned_to_floats_only():
    # hidden_dump is a float pointer: 4, 8 and 12 bytes past a 16-byte boundary it takes the same rows, and nothing beside them
    import torch
    from paper_2503_08524_amd import binding
    s = ModelShape("dump", L=2, d=256, H=2, H_kv=2, hd=128, F=384, V=512, dtype="bf16")
    dec = binding.Decoder(s, binding.random_weights_on_device(s, 5), 3, 40)
    toks = torch.from_numpy(d3_inputs.make_prompt(3, 40, s.V, seed=1)).to("cuda:0")
    n = (s.L + 1) * 3 * s.d
    want = torch.zeros(n, device="cuda:0")
    print("case hidden_dump alignment", flush=True)
    dec.prefill(toks, hidden_dump=want)
    for off in (1, 2, 3):
        buf = torch.full((n + 8,), 7.0, device="cuda:0")
        dec.prefill(toks, hidden_dump=buf[off:off + n])
        assert torch.equal(buf[off:off + n], want) and bool((buf[:off] == 7).all()) and bool((buf[off + n:] == 7).all())
    dec.close()


@pytest.mark.parametrize("ks", [2, 3, 4])
def test_prompt_residual_projections_in_k_parts(monkeypatch, ks):
    # the projections of a prompt pass with K cut into 2, 3 and 4 parts (one workgroup each), which takes two whole stages for
    # every part (contractions too short for that stay whole): K of 8 stages (QKV, gate/up), 16 (O) and 21.5 (down; uneven parts, the last
    # with the stages over); at head_dim 64 8 and 11 stages; then 4 and 11, where 3 and 4 parts cut the down projection alone.  By itself the
    # launcher cuts K only for long contractions (the 7B / 13B / 70B widths, which the all-block and full-size tests run)
    monkeypatch.setenv("D3_PROMPT_KS", str(ks))
    _run(SMALL_GQA, 1, 300, 3, 0.8, 1, forced_seed=21)
    _run(ModelShape("parts-hd64", L=2, d=512, H=8, H_kv=8, hd=64, F=704, V=512, dtype="bf16"), 2, 200, 3, 0.9, 1, forced_seed=21)
    _run(SMALL_BF16, 2, 200, 3, 0.9, 2, forced_seed=21)


def test_every_projection_in_the_most_k_parts(monkeypatch):
    # 16 stages (QKV, O, gate/up) and 17.5 (down) in 8 parts: one pair of stages each, the last of the down projection with the stages over
    monkeypatch.setenv("D3_PROMPT_KS", "8")
    s = ModelShape("most-parts", L=2, d=1024, H=8, H_kv=2, hd=128, F=1120, V=512, dtype="bf16")
    gpu, gens = _run(s, 1, 150, 2, 1.0, 1, forced_seed=21, kv_dtype="f32")
    helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


def test_lds_tiled_prompt_kernel_shapes():
    # rows that do not fill the last row block (d_ffn 1376 = 10.75 blocks of 128 gate/up pairs, vocab 2000), five and a half
    # column blocks; K of 8 stages and of 21.5 (10 pairs, then a whole and a half stage one at a time); then head_dim 64
    # (vector-ALU attention per column) with 1100 tokens, K of 4 and 11 stages
    _run(SMALL_GQA, 1, 700, 3, 0.8, 1, forced_seed=19)
    _run(SMALL_BF16, 1, 1100, 3, 0.9, 2, forced_seed=19)
    # the shortest contractions: K of one pair of stages (prologue and tail) and of three stages
    _run(ModelShape("narrow", L=2, d=128, H=2, H_kv=1, hd=64, F=192, V=512, dtype="bf16"), 1, 300, 3, 0.9, 1, forced_seed=19)


@pytest.mark.parametrize("d,F,P,ks", [(128, 128, 129, 0), (160, 224, 255, 0), (192, 352, 257, 1), (256, 608, 384, 2), (512, 1120, 130, 3),
                                      (288, 96, 140, 0), (512, 2048, 513, 8)])
def test_prompt_kernel_contractions_and_parts(monkeypatch, d, F, P, ks):
    # the LDS-tiled kernel walks K in pairs of 64-wide stages: contractions that are one pair, that leave 32, 64 and 96 over,
    # that are too short for it (96: the panel kernel in blocks of 64 columns), and K parts of uneven length where the contraction has two
    # whole stages for every part (8 parts: the down projection's 32 stages alone); column blocks of 1, 2, 127 and 128 live columns.  Rows of the last row block are missing throughout.  With an fp32 cache only fp32 sums and the 16 bits
    # of an activation's two bf16 halves are left: 2^-17 per product, far below the bound of 1e-4.
    if ks:
        monkeypatch.setenv("D3_PROMPT_KS", str(ks))
    s = ModelShape("odd-k", L=2, d=d, H=2, H_kv=1, hd=128, F=F, V=512, dtype="bf16")
    gpu, gens = _run(s, 1, P, 2, 1.0, 1, forced_seed=19, kv_dtype="f32")
    helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("P,blocks", [(65, 1), (100, 2), (128, 4)])
def test_short_prompts_on_the_prompt_kernel(monkeypatch, P, blocks):
    # 65 to 128 columns: the LDS-tiled kernel takes the projections with enough row blocks (all, then gate/up and QKV, then gate/up
    # alone), the panel kernel the others; each reads the other's partial sums of squares and activations
    monkeypatch.setenv("D3_PROMPT_ROW_BLOCKS", str(blocks))
    s = ModelShape("short", L=2, d=256, H=2, H_kv=1, hd=128, F=608, V=512, dtype="bf16")
    gpu, gens = _run(s, 1, P, 2, 1.0, 1, forced_seed=19, kv_dtype="f32")
    helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("cus,F,P", [(4, 2048, 700), (7, 2080, 1100), (4, 2144, 513), (7, 4096, 900)])
def test_prompt_tiles_whole_and_in_parts_in_one_launch(monkeypatch, cus, F, P):
    # the down projection's row block x 5 to 9 column blocks, in rounds of 4 or 7 tiles: whole tiles first, then 1 or 2 tiles in 2 to 5
    # parts each, of 32 stages and of 32.5, 33.5 and 64 (uneven parts, single stages in the last)
    monkeypatch.setenv("D3_PROMPT_CUS", str(cus))
    s = ModelShape("mixed", L=2, d=256, H=2, H_kv=1, hd=128, F=F, V=512, dtype="bf16")
    gpu, gens = _run(s, 1, P, 2, 1.0, 1, forced_seed=19, kv_dtype="f32")
    helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("cus,d,F,P", [(4, 2048, 384, 300), (7, 2048, 512, 400), (5, 4096, 640, 300), (4, 2080, 384, 300)])
def test_storing_projections_whole_and_in_parts_in_one_launch(monkeypatch, cus, d, F, P):
    # QKV (two row blocks) and gate/up (3 to 5) x 3 or 4 column blocks in rounds of 4, 5 or 7 tiles: whole tiles, which store everything, and in the
    # same launch tiles in parts, which store a share each: QKV 1 or 2 tiles in 2, 4 and 5 parts, gate/up in 3 and 4 (and whole tiles alone); 32 stages,
    # 64, and 32.5 with the half stage in the last part
    monkeypatch.setenv("D3_PROMPT_CUS", str(cus))
    s = ModelShape("mixed-store", L=2, d=d, H=2, H_kv=1, hd=128, F=F, V=512, dtype="bf16")
    gpu, gens = _run(s, 1, P, 2, 1.0, 1, forced_seed=19, kv_dtype="f32")
    helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("ks", [3, 5, 6, 7])
def test_parts_that_finish_several_runs_together(monkeypatch, ks):
    # QKV (four row blocks) and gate/up (five) of one column block, every tile in 3 to 7 parts with 8 units between them: runs of one to three units,
    # on both sides of the two column tiles, of which the part that comes last takes all that wait for it; 16 stages
    monkeypatch.setenv("D3_PROMPT_KS", str(ks))
    monkeypatch.setenv("D3_PROMPT_ROW_BLOCKS", "1")
    s = ModelShape("runs", L=2, d=1024, H=4, H_kv=2, hd=128, F=640, V=512, dtype="bf16")
    gpu, gens = _run(s, 1, 100, 2, 1.0, 1, forced_seed=19, kv_dtype="f32")
    helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


# cus: compute units that the launches reckon with (8 workgroups at least).  K of 4 stages, the fewest (whole tiles, dead rows and columns in the last); 7 row blocks x 3
# column blocks of 5 stages in three rounds; tiles left over in parts: QKV and gate/up (two and five row blocks) of 64 stages, 4, 6, 10 and 2 tiles on 8 and 16
# workgroups, i.e. mains with one helper, with two and three, helpers with pieces of several tiles, and tiles behind a full round; down of 64 and 172 stages, one
# row block, in parts of uneven length, up to the most there are
LARGE_TILES = [(0, 256, 320, 300, "f16"), (8, 320, 832, 700, "f32"), (8, 4096, 640, 300, "f32"), (8, 4096, 640, 513, "f16"), (16, 4096, 1280, 256, "f32"),
               (8, 256, 4096, 700, "f32"), (16, 256, 11008, 600, "f32"), (8, 256, 11008, 1100, "f32")]


@pytest.mark.parametrize("cus,d,F,P,kv", LARGE_TILES)
def test_prompt_tiles_of_256_columns(monkeypatch, cus, d, F, P, kv):
    monkeypatch.setenv("D3_PROMPT_TILE", "256")
    if cus:
        monkeypatch.setenv("D3_PROMPT_CUS", str(cus))
    s = ModelShape("large-tiles", L=2, d=d, H=2, H_kv=1, hd=128, F=F, V=512, dtype="bf16")
    gpu, gens = _run(s, 1, P, 2, 1.0, 1, forced_seed=19, kv_dtype=kv)
    if kv == "f32":
        helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)
    else:
        helpers.compare(gpu, gens, 2)


# passes in lines by the estimate, whose other projections take the smaller tiles: of 128 columns, and head_dim 64, whose QKV rotates in a launch of its own
@pytest.mark.parametrize("d,H,H_kv,hd,F,P", [(1024, 8, 8, 128, 2816, 1536), (2048, 32, 8, 64, 8192, 812)])
def test_passes_with_tiles_of_both_sizes(d, H, H_kv, hd, F, P):
    s = ModelShape("both-tiles", L=1, d=d, H=H, H_kv=H_kv, hd=hd, F=F, V=512, dtype="bf16")
    gpu, gens = _run(s, 1, P, 2, 1.0, 0, forced_seed=19, kv_dtype="f16")
    helpers.compare(gpu, gens, 2)


# one prompt, a last token by itself, prompts that share passes, unequal ones
@pytest.mark.parametrize("B,P,lengths", [(1, 2056, None), (1, 2049, None), (2, 1030, None), (2, 1100, (1100, 950))])
def test_few_columns_behind_2048_are_a_pass_of_their_own(monkeypatch, B, P, lengths):
    # bit for bit what passes of 2048 columns give
    import torch
    from paper_2503_08524_amd import binding
    s = ModelShape("few-behind", L=2, d=256, H=2, H_kv=2, hd=128, F=512, V=512, dtype="bf16")
    w, toks = binding.random_weights_on_device(s, 5), torch.from_numpy(d3_inputs.make_prompt(B, P, s.V, seed=1)).to("cuda:0")
    got = []
    print(f"case few columns behind 2048, B={B} P={P}", flush=True)
    for cols in (None, "2048"):
        monkeypatch.setenv("D3_PREFILL_COLS", cols) if cols else monkeypatch.delenv("D3_PREFILL_COLS", raising=False)
        dec, logits = binding.Decoder(s, w, B, P, kv_dtype="f16"), torch.zeros(B, s.V, device="cuda:0")
        dec.prefill_ragged(toks, list(lengths), logits=logits) if lengths else dec.prefill(toks, logits=logits)
        torch.cuda.synchronize()
        got.append((logits, dec.k_cache.clone(), dec.v_cache.clone()))
        dec.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))


def test_fp32_caches_keep_the_tiles_that_sum_in_two_accumulators(monkeypatch):
    # the pass above with an fp32 cache, whose rounding does not hide twice as many roundings in a row: bit for bit what the smaller tiles give
    import torch
    from paper_2503_08524_amd import binding
    s = ModelShape("fp32-cache", L=2, d=1024, H=8, H_kv=8, hd=128, F=2816, V=512, dtype="bf16")
    w, toks = binding.random_weights_on_device(s, 5), torch.from_numpy(d3_inputs.make_prompt(1, 1536, s.V, seed=1)).to("cuda:0")
    got = []
    print("case fp32 cache", flush=True)
    for tile in (None, "128", "256"):
        monkeypatch.setenv("D3_PROMPT_TILE", tile) if tile else monkeypatch.delenv("D3_PROMPT_TILE", raising=False)
        dec, logits = binding.Decoder(s, w, 1, 1536, kv_dtype="f32"), torch.zeros(1, s.V, device="cuda:0")
        dec.prefill(toks, logits=logits)
        torch.cuda.synchronize()
        got.append((logits, dec.k_cache.clone(), dec.v_cache.clone()))
        dec.close()
    assert all(torch.equal(a, b) for a, b in zip(got[0], got[1]))
    assert not torch.equal(got[1][1], got[2][1])       # the larger tiles' sums do differ


def test_prompt_tiles_of_256_columns_replay_from_a_graph(monkeypatch):
    # tiles in parts leave their arrival counters zero: each replay, on new tokens in between, equals the eager call bit for bit; two sequences that share passes
    import torch
    from paper_2503_08524_amd import binding
    monkeypatch.setenv("D3_PROMPT_TILE", "256")
    monkeypatch.setenv("D3_PROMPT_CUS", "8")
    s = ModelShape("graph-256", L=2, d=2048, H=2, H_kv=1, hd=128, F=4096, V=512, dtype="bf16")
    B, P = 2, 350
    dec = binding.Decoder(s, binding.random_weights_on_device(s, 5), B, P + 2)
    toks = [torch.from_numpy(d3_inputs.make_prompt(B, P, s.V, seed=k)).to("cuda:0") for k in (1, 2)]
    fed, out, logits = toks[0].clone(), torch.zeros(B, dtype=torch.int32, device="cuda:0"), torch.zeros(B, s.V, device="cuda:0")
    print("case graph of tiles of 256 columns", flush=True)
    want = []
    for t in toks:
        dec.prefill(t, next_tok=out, logits=logits)
        want.append((out.clone(), logits.clone(), dec.k_cache.clone()))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dec.prefill(fed, next_tok=out, logits=logits)
    for k in (0, 1, 1, 0, 1):
        fed.copy_(toks[k])
        logits.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[k][0]) and torch.equal(logits, want[k][1]) and torch.equal(dec.k_cache, want[k][2])
    dec.close()


@pytest.mark.parametrize("ks", [1, 2])
def test_prompt_projection_rotates_with_two_stated_roundings(monkeypatch, ks):
    # 200 times the same token: every position has the same unrotated key, which position 0 (cos 1, sin 0) shows, so the rotated ones follow
    # bit by bit from fma(lo, cos, -(hi sin)), fma(lo, sin, hi cos) over the table's floats.  The products are exact in float64; rounding their sum
    # to float64 first, or a cosine that two libraries round to neighbouring floats, is left to one element in a thousand.
    import torch
    from paper_2503_08524_amd import binding
    monkeypatch.setenv("D3_PROMPT_KS", str(ks))
    P, hd = 200, 128
    s = ModelShape("rotate", L=1, d=256, H=2, H_kv=1, hd=hd, F=256, V=512, dtype="bf16")
    dec = binding.Decoder(s, binding.weights_to_device(s, d3_inputs.make_weights(s, 3), "cuda:0"), 1, P + 1, kv_dtype="f32")
    print(f"case rotate ks={ks}", flush=True)
    dec.prefill(torch.full((1, P), 7, dtype=torch.int32, device="cuda:0"))
    torch.cuda.synchronize()
    k = dec.k_cache[0, 0, 0, :P].cpu().numpy()
    dec.close()
    lo, hi = k[0, :hd // 2], k[0, hd // 2:]
    angle = np.arange(P)[:, None] * s.rope_base ** (-2.0 * np.arange(hd // 2) / hd)
    cs, sn = np.cos(angle).astype(np.float32), np.sin(angle).astype(np.float32)
    exact = lambda a, b: a.astype(np.float64) * b.astype(np.float64)
    y0 = (exact(lo, cs) - (hi * sn).astype(np.float64)).astype(np.float32)
    y1 = (exact(lo, sn) + (hi * cs).astype(np.float64)).astype(np.float32)
    assert np.mean(np.concatenate([y0, y1], 1) != k) <= 1e-3


@pytest.mark.parametrize("F,P,split_mb", [(512, 130, 300), (2560, 70, 300), (2560, 70, 1)])
def test_prompt_kernel_adds_up_many_partial_sums_of_squares(monkeypatch, F, P, split_mb):
    # a column's sum of squares in more partials than one read of 16 threads takes: 130 columns, which all projections take to the LDS-tiled kernel: the
    # 18 row blocks of its own O and down.  70 columns, where 18 row blocks stay with the panel kernel and the 20 of gate/up do not, by the line pinned
    # here: the 72 row groups of one launch (four waves of one row tile), or the 36 of two launches of 64 columns (eight waves, one row tile pinned).
    monkeypatch.setenv("D3_PROMPT_ROW_BLOCKS", "20")
    monkeypatch.setenv("D3_WIDE_SPLIT_MB", str(split_mb))
    monkeypatch.setenv("D3_WIDE_RT", "1")
    s = ModelShape("many-parts", L=2, d=4608, H=2, H_kv=1, hd=128, F=F, V=512, dtype="bf16")
    gpu, gens = _run(s, 1, P, 2, 1.0, 1, forced_seed=19, kv_dtype="f32")
    helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("rt", [1, 2, 4])
@pytest.mark.parametrize("d,F,B,P", [(8192, 256, 3, 2), (8192, 256, 12, 1), (256, 12288, 2, 5)])
def test_rows_begun_at_different_places_by_every_number_of_row_tiles(monkeypatch, d, F, B, P, rt):
    # QKV, gate/up and lm_head over K = 8192 with 3 (packed) and 12 columns, down over K = 12288 with 2 and 5 of a prompt, with 1, 2 and 4 row
    # tiles a wave (gate/up: 1 and 2 pairs), the largest that is at most the one pinned
    monkeypatch.setenv("D3_MFMA_RT", str(rt))
    s = ModelShape("far-rows", L=1, d=d, H=2, H_kv=1, hd=128, F=F, V=512, dtype="bf16")
    gpu, gens = _run(s, B, P, 2, 1.0, 0, forced_seed=19, kv_dtype="f32")
    helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("d,F,B,P", [(8192, 256, 3, 2), (8192, 256, 12, 1), (12288, 256, 20, 1), (256, 12288, 2, 20), (256, 12288, 1, 40)])
def test_rows_a_multiple_of_8_kb_apart(d, F, B, P):
    # batched projections whose workgroups begin their rows at different places: QKV, gate/up and lm_head over K = 8192 with 3 (packed) and 12
    # columns and over K = 12288 with 20 (panel kernel, 8 slices of 12 turns), the down projection over K = 12288 with 2, 20 shared and 40 columns.
    # Only fp32 sums and the 16 bits of an activation's two bf16 halves are left with an fp32 cache.
    s = ModelShape("far-rows", L=1, d=d, H=2, H_kv=1, hd=128, F=F, V=512, dtype="bf16")
    gpu, gens = _run(s, B, P, 2, 1.0, 0, forced_seed=19, kv_dtype="f32")
    helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("dtype,d,F,B", [("f32", 64, 15360, 1), ("bf16", 64, 15360, 1), ("f32", 3840, 64, 4), ("f32", 3072, 64, 3), ("f32", 64, 7680, 2), ("f32", 2816, 3840, 4)])
def test_vector_alu_gemv_with_most_lds(dtype, d, F, B):
    # as many columns as an input's LDS budget of 60 KB takes, beside which every column count keeps its finished units: 66, 70 and 78 KB a workgroup, and
    # the first width at which four columns pass 64 KB
    s = ModelShape("gemv-lds", L=1, d=d, H=1, H_kv=1, hd=64, F=F, V=256, dtype=dtype)
    gpu, gens = _run(s, B, 3, 3, 1.0, 0, forced_seed=19, kv_dtype="f32")
    helpers.compare(gpu, gens, 3, logit_atol=1e-4, hidden_tol=1e-5)


@pytest.mark.parametrize("d,B", [(1408, 1), (1408, 3), (64, 1), (4160, 1)])
def test_infinite_gain_stays_out_of_the_padding(d, B):
    # an infinite gain of the last element makes every logit infinite, with the sign of that element times its weight, and none of them no number:
    # what fills the last stride of a row is zero, whatever the gains (fp32: rows of 5.5, 0.25 and 16.25 strides)
    import torch
    from paper_2503_08524_amd import binding
    s = ModelShape("inf-gain", L=1, d=d, H=1, H_kv=1, hd=64, F=64, V=512, dtype="f32")
    w = binding.weights_to_device(s, d3_inputs.make_weights(s, 3), "cuda:0")
    w["final_norm"][d - 1] = float("inf")
    dec = binding.Decoder(s, w, B, 8, kv_dtype="f32")
    lg, hid = torch.empty(B, s.V, device="cuda:0"), torch.empty(2, B, d, device="cuda:0")
    print(f"case inf-gain d={d} B={B}", flush=True)
    dec.prefill(torch.from_numpy(d3_inputs.make_prompt(B, 1, s.V, seed=5)).to("cuda:0"), logits=lg, hidden_dump=hid)
    want = torch.sign(hid[1, :, d - 1:] * w["lm_head"][:, d - 1]) * float("inf")
    assert torch.equal(lg, want)
    dec.close()


@pytest.mark.parametrize("dtype,H", [("bf16", 64), ("f32", 32)])
def test_rows_of_16_kb_stream_as_fast_as_others(dtype, H):
    # the O projection at batch 1, square: rows of 16 KB (a power of two) against rows one head longer, four blocks of each.  The rate of either differs by a
    # few per cent from run to run; waves that meet on a part of the memory channels cost a fifth of it.  Best of eight readings of each.
    import torch
    from paper_2503_08524_amd import binding

    def rate(heads):
        s = ModelShape("rows", L=4, d=heads * 128, H=heads, H_kv=heads, hd=128, F=64, V=64, dtype=dtype)
        wt = torch.bfloat16 if dtype == "bf16" else torch.float32
        new = lambda r, c: torch.empty(r, c, device="cuda:0").normal_(0, 0.02).to(wt)
        gain = torch.ones(s.d, device="cuda:0")
        kv = s.H_kv * s.hd
        w = {"tok_emb": new(s.V, s.d), "lm_head": new(s.V, s.d), "final_norm": gain, "layers": [
            {"attn_norm": gain, "wq": new(s.d, s.d), "wk": new(kv, s.d), "wv": new(kv, s.d), "wo": new(s.d, s.d), "mlp_norm": gain,
             "w_gate": new(s.F, s.d), "w_up": new(s.F, s.d), "w_down": new(s.d, s.F)} for _ in range(s.L)]}
        dec = binding.Decoder(s, w, 1, 64, kv_dtype="f32")
        tok = dec.prefill(torch.ones(1, 4, dtype=torch.int32, device="cuda:0"))
        out, best = torch.empty_like(tok), 0.0
        dec.set_plan_table([s.L, s.L], [0, 0])
        dec.profile_select(binding.D3_K_OPROJ)
        for _ in range(9):
            for _ in range(10):
                dec.truncate(4)
                dec.decode_step(tok, 1, out)
            ms, n = dec.profile_read()
            best = max(best, s.d * s.d * w["lm_head"].element_size() * n / ms / 1e9)
        dec.close()
        return best

    plain, odd = rate(H), rate(H + 1)
    print(f"case rows {dtype}: 16 KB {plain:.2f} TB/s, longer {odd:.2f} TB/s", flush=True)
    assert plain > 0.9 * odd


@pytest.mark.parametrize("d,F,V,B", [(64, 64, 270016, 1), (64, 4160, 512, 2), (1408, 64, 512, 3)])
def test_vector_alu_gemv_strides_and_units(d, F, V, B):
    # rows of one 64-lane stride, of 16 and a quarter and of five and a half, begun at every stride of a row; one more than a wave's fill of units per wave,
    # which takes more workgroups than the launch would have (135008 pairs of rows against 2048 waves of 64)
    s = ModelShape("gemv", L=2, d=d, H=1, H_kv=1, hd=64, F=F, V=V, dtype="f32")
    gpu, gens = _run(s, B, 3, 3, 1.0, 1, forced_seed=19, kv_dtype="f32")
    helpers.compare(gpu, gens, 3, logit_atol=1e-4, hidden_tol=1e-5)


@pytest.mark.parametrize("B", [1, 2])
@pytest.mark.parametrize("H,H_kv,kv,P", [(2, 2, "f16", 130), (2, 2, "f16", 257), (3, 3, "f32", 65), (4, 2, "f16", 193), (4, 2, "f32", 129),
                                         (8, 2, "f16", 161), (8, 1, "f16", 150), (8, 1, "f32", 97), (8, 8, "f16", 64)])
def test_prompt_attention_over_the_whole_context(monkeypatch, H, H_kv, kv, P, B):
    # the kernel of long prompt chunks (128 (query, head) pairs per workgroup), forced on short ones, one sequence or two: group sizes 1, 2, 4 and 8, KV heads that
    # do and do not divide over the XCDs, last query tiles of 1 to 128 pairs, row tiles (64 rows fp16, 32 fp32) that end on, before
    # and past a boundary, one and several steps of the two wave groups, and a group that sees no row of some entries
    monkeypatch.setenv("D3_PROMPT_ATTN_WGS", "1")
    s = ModelShape("prompt-attn", L=2, d=256, H=H, H_kv=H_kv, hd=128, F=384, V=512, dtype="bf16")
    gpu, gens = _run(s, B, P, 2, 1.0, 1, forced_seed=19, kv_dtype=kv)
    if kv == "f32":     # only arithmetic rounding is left (16 bits of an activation's two bf16 halves, 21 of the fp16 pairs)
        helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("B,P,H,H_kv,cols,lengths,kv", [(2, 37, 2, 2, 0, None, "f32"), (3, 150, 4, 2, 256, None, "f16"), (2, 700, 4, 1, 512, None, "f32"),
                                                         (5, 19, 8, 1, 0, None, "f16"), (4, 300, 4, 2, 256, (300, 1, 37, 2), "f32"),
                                                         (3, 700, 8, 1, 320, (129, 700, 66), "f16"), (2, 260, 3, 3, 128, (65, 260), "f32")])
def test_shared_passes_with_query_tiles_run_by_run(monkeypatch, B, P, H, H_kv, cols, lengths, kv):
    # what short turns behind long caches take, forced on prompts: the query-tile kernel, a launch per sequence of a shared pass, over
    # its own columns of q and of the outputs, with the context split where it is long; group sizes 1, 2, 4 and 8, passes that end inside a
    # sequence, runs of one column, sequences that begin inside a later split (left-padded batches)
    monkeypatch.setenv("D3_PROMPT_ATTN_WGS", str(1 << 20))
    if cols:
        monkeypatch.setenv("D3_PREFILL_COLS", str(cols))
    s = ModelShape("by-run", L=2, d=256, H=H, H_kv=H_kv, hd=128, F=384, V=512, dtype="bf16")
    gpu, gens = _run(s, B, P, 2, 1.0, 1, forced_seed=19, kv_dtype=kv, lengths=None if lengths is None else np.array(lengths, np.int32), max_seq=P + 2)
    if kv == "f32":     # only arithmetic rounding is left
        helpers.compare(gpu, gens, 2, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("kv,past,n,launches", [("f16", 4096, 16, 2), ("f32", 4096, 16, 2), ("f16", 64, 16, 1), ("f16", 4096, 1000, 1)])
def test_short_turns_behind_a_long_cache_split_their_context(monkeypatch, kv, past, n, launches):
    # the whole-context kernel walks a cache of 4096 rows in 32 (fp16) or 64 (fp32) steps on the two workgroups that 16 tokens make, so these
    # turns take the query tiles with a split context, one launch per sequence and block; a short cache or a long turn takes one launch.
    # Either route computes the same: the bound is that of the fp32-cache cases here, with an fp16 cache its 11 bits.
    import torch
    from paper_2503_08524_amd import binding
    s = ModelShape("long-cache", L=2, d=256, H=4, H_kv=2, hd=128, F=384, V=512, dtype="bf16")
    w = binding.random_weights_on_device(s, 3)
    toks = torch.from_numpy(d3_inputs.make_prompt(2, past + n, s.V, seed=1)).to("cuda:0")
    print(f"case {n} tokens behind {past} rows, kv={kv}", flush=True)
    got = []
    for wgs in (None, 1, 1 << 20):
        if wgs:
            monkeypatch.setenv("D3_PROMPT_ATTN_WGS", str(wgs))
        dec = binding.Decoder(s, w, 2, past + n, kv_dtype=kv)
        dec.prefill(toks[:, :past].contiguous())
        logits = torch.zeros(2, s.V, dtype=torch.float32, device="cuda:0")
        dec.profile_select(binding.D3_K_ATTN)
        dec.prefill(toks[:, past:].contiguous(), pos_begin=past, logits=logits)
        got.append((dec.profile_read()[1] / s.L, logits))
        dec.close()
    assert [k for k, _ in got] == [launches, 1, 2]
    for _, other in got[1:]:
        assert float((got[0][1] - other).abs().max()) <= (2e-4 if kv == "f32" else 5e-3)


@pytest.mark.parametrize("B,kv", [(1, "f16"), (3, "f16"), (2, "f32")])
def test_small_gqa(B, kv):
    _run(SMALL_GQA, B, 37, 6, 0.8, 1, forced_seed=8, kv_dtype=kv)


@pytest.mark.parametrize("B,P", [(2, 300), (1, 700)])
def test_fp32_cache_on_the_matrix_core_attention_kernels(B, P):
    # grouped-query attention at head_dim 128 with an fp32 cache (what models deeper than 48 blocks get): the cache rows go
    # to the matrix cores as fp16 hi + lo planes; prompts of 2 x 300 columns in one pass (whole context) and of 700 (query tiles), decode contexts
    # that span three and six splits, batch 1 (vector-ALU projections) and batch 2 (matrix-core projections).  The fp32
    # rows leave nothing but arithmetic rounding: the logits must agree 100 times closer than the acceptance bound.
    gpu, gens = _run(SMALL_GQA, B, P, 5, 0.8, 1, forced_seed=8, kv_dtype="f32")
    helpers.compare(gpu, gens, 5, logit_atol=2e-4, hidden_tol=1e-4)


@pytest.mark.parametrize("kv", ["f16", "f32"])
def test_batch1_decode_grouped_query_head_dim_128(kv):
    _run(SMALL_GQA, 1, 70, 12, 0.85, 1, forced_seed=14, kv_dtype=kv)


@pytest.mark.parametrize("B,hd,H,H_kv,kv", [(1, 128, 4, 2, "f32"), (3, 128, 4, 2, "f32"), (2, 64, 8, 2, "f16"), (2, 64, 8, 1, "f16"), (3, 64, 4, 4, "f16")])
def test_vector_alu_attention_over_several_splits(B, hd, H, H_kv, kv):
    # pairs of heads over fp32 rows of 128 (three workgroups per compute unit), and rows of eight lanes, whose maxima go through the LDS: 4 splits
    s = ModelShape("splits", L=2, d=256, H=H, H_kv=H_kv, hd=hd, F=256, V=512, dtype="bf16")
    gpu, gens = _run(s, B, 400, 3, 1.0, 1, forced_seed=19, kv_dtype=kv)
    if kv == "f32":
        helpers.compare(gpu, gens, 3, logit_atol=2e-4, hidden_tol=1e-4)


def test_batch1_zero_blocks_and_free_running_tokens():
    gpu, gens = _run(SMALL_GQA, 1, 9, 6, 0.5, 1)      # keep = 3, 1, 0, 0, ...: steps with no block at all
    assert gens[0].keep[2] == 0


def test_long_context_spans_several_attention_splits():
    _run(SMALL_BF16, 2, 700, 4, 0.9, 2, forced_seed=9)


def test_window_at_block_zero_and_min_keep():
    _run(SMALL_BF16, 2, 5, 10, 0.7, 0, forced_seed=10, min_keep=1)


def test_zero_blocks_kept():
    # alpha = 0.5 on 4 blocks: keep = 4, 2, 1, 0, 0: the last steps run the embedding and lm_head only
    _run(SMALL_BF16, 1, 4, 5, 0.5, 1, forced_seed=11)


def test_llama7b_widths_two_blocks_batch1():
    _run(d3_inputs.LLAMA_7B.truncated(2), 1, 8, 5, 0.7, 1, forced_seed=12)


def test_llama7b_widths_two_blocks_batch4():
    _run(d3_inputs.LLAMA_7B.truncated(2), 4, 3, 3, 0.7, 1, forced_seed=13)


def test_llama13b_widths_one_block_batch4():
    # 13B widths, batch 4: the matrix-core path with one column tile at real K (5120 / 13824) and row counts
    _run(d3_inputs.LLAMA_13B.truncated(1), 4, 2, 3, 1.0, 0, forced_seed=15)


def test_llama70b_widths_one_block_gqa():
    # 70B widths: grouped-query attention (64 query / 8 KV heads) and d_ffn 28672, which only the matrix-core
    # path can take (batch 1 included); one set of weights serves both batch sizes
    shape = d3_inputs.LLAMA_70B.truncated(1)
    w = d3_inputs.make_weights(shape, 0)
    for B in (2, 1):
        prompts = d3_inputs.make_prompt(B, 2, shape.V, seed=1)
        forced = _forced(B, 2, shape.V, 16)
        print(f"case {shape.name} B={B}", flush=True)
        gpu = helpers.gpu_generate(shape, w, prompts, 2, 1.0, 0, forced=forced)
        _, gens = helpers.oracle_generate(shape, w, prompts, 2, 1.0, 0, forced=forced)
        wl, wh = helpers.compare(gpu, gens, 2)
        print(f"  worst logit abs err {wl:.3e}, worst hidden rel L2 {wh:.3e}", flush=True)
        del gpu


def test_full_size_7b_configuration_sampled_against_oracle():
    """The benchmark's own launch configuration (7B shape, 32 blocks, batch 1, prompt 512) checked on the
    outputs the oracle can afford: the hidden state after block 0 of the last prompt position and of every
    decode step, and the complete logits of the steps that keep only block 0 / no block (alpha = 0.5 keeps
    32, 16, 8, 4, 2, 1, 0 blocks).  All 32 blocks point at the same weight tensors, so the host draws one
    block; the oracle runs that block alone over the 518 rows."""
    import torch
    from oracle import oracle
    from paper_2503_08524_amd import binding

    full = d3_inputs.LLAMA_7B
    one = full.truncated(1)
    w1 = d3_inputs.make_weights(one, 0)
    w_tied = dict(w1)
    w_tied["layers"] = [w1["layers"][0]] * full.L
    P, G, alpha, start = 512, 7, 0.5, 19
    prompts = d3_inputs.make_prompt(1, P, full.V, seed=1)
    forced = _forced(1, G, full.V, 17)
    keep, drop, ids = binding.d3_plan_depth(full.L, alpha, start, 0, G)
    assert keep.tolist() == [32, 16, 8, 4, 2, 1, 0] and ids[5, 0] == 0

    # GPU: the real thing, one device copy of the block shared by all 32 layer entries
    dev = binding.weights_to_device(one, w1)
    dev_tied = dict(dev)
    dev_tied["layers"] = [dev["layers"][0]] * full.L
    dec = binding.Decoder(full, dev_tied, 1, P + G)
    print("case full-size 7B, tied blocks", flush=True)
    gpu = helpers.gpu_generate(full, None, prompts, G, alpha, start, forced=forced, decoder=dec, fill_each_step=True)

    # oracle: block 0 alone over every row
    oracle.set_threads(helpers.oracle_threads())
    model = oracle.OracleModel(one, w1)
    seq = model.new_seq(P + G)
    hid = None
    for p in range(P):
        hid, _ = seq.forward_token(int(prompts[0, p]), p, [0], want_hidden=(p == P - 1))
    def rel(a, b):
        return float(np.linalg.norm(a - b) / np.linalg.norm(b))
    assert rel(gpu["hidden"][0][1, 0].astype(np.float64), hid[1]) <= helpers.HIDDEN_REL_L2
    worst = 0.0
    for i in range(1, G):
        blocks = [0] if keep[i] >= 1 else []
        h, lg = seq.forward_token(int(forced[0, i - 1]), P + i - 1, blocks, want_hidden=True, want_logits=True)
        got = gpu["hidden"][i][:, 0].astype(np.float64)
        assert rel(got[0], h[0]) <= 1e-6                                   # the embedding row
        if keep[i] >= 1:
            assert rel(got[1], h[1]) <= helpers.HIDDEN_REL_L2, f"step {i}"
        if keep[i] <= 1:                                                    # logits depend on block 0 at most
            err = float(np.abs(gpu["logits"][i][0].astype(np.float64) - lg).max())
            worst = max(worst, err)
            assert err <= helpers.LOGIT_ATOL, f"step {i}: logits max abs err {err:.3e}"
            top2 = np.partition(lg, -2)[-2:]
            if top2[1] - top2[0] > helpers.TOKEN_MARGIN:
                assert int(gpu["tokens"][i][0]) == oracle.argmax(lg)
    print(f"  worst logit abs err {worst:.3e}", flush=True)
    # the fill of the dropped blocks copied the source block's rows (bit-exact), at full cache size
    for i in (1, 5):
        pos, s, n = P + i - 1, int(drop[i]), full.L - int(keep[i])
        src = s - 1
        assert torch.equal(dec.k_cache[s, 0, :, pos], dec.k_cache[src, 0, :, pos])
        assert torch.equal(dec.v_cache[s + n - 1, 0, :, pos], dec.v_cache[src, 0, :, pos])


@pytest.mark.timeout(400)
@pytest.mark.parametrize("name,B,P", [("llama-13b", 4, 1024), ("llama-7b", 32, 2048), ("llama-70b", 8, 1024)])
def test_full_size_batched_configurations_sampled_against_oracle(name, B, P):
    """The batched benchmark configurations in their own launch configuration (all blocks, full batch, full prompt),
    checked on what the oracle can afford for two sampled sequences (the first and the last of the batch): the hidden
    state after block 0 of the last prompt position and of every decode step, and the complete logits of the steps that
    keep only block 0 / no block (alpha = 0.5 halves the depth every step).  All blocks point at the same weight
    tensors, so the host draws one block.  For a sampled sequence the oracle fills block 0's cache rows of the prompt
    with its cache-write-only entry (those rows depend on the embeddings alone) and runs block 0 in full for the rows
    that are compared."""
    import torch
    from oracle import oracle
    from paper_2503_08524_amd import binding

    full = d3_inputs.SHAPES[name]
    one = full.truncated(1)
    w1 = d3_inputs.make_weights(one, 0)
    alpha, start = 0.5, d3_inputs.start_layer_from_fraction(full.L, 0.6)
    G = int(np.floor(np.log2(full.L))) + 2                       # depth L, L/2, ..., 1, 0
    keep, drop, ids = binding.d3_plan_depth(full.L, alpha, start, 0, G)
    assert keep[0] == full.L and keep[G - 2] == 1 and keep[G - 1] == 0 and all(ids[i, 0] == 0 for i in range(G - 1))
    prompts = d3_inputs.make_prompt(B, P, full.V, seed=1)
    forced = _forced(B, G, full.V, 17)

    dev = binding.weights_to_device(one, w1)
    dev_tied = dict(dev)
    dev_tied["layers"] = [dev["layers"][0]] * full.L
    dec = binding.Decoder(full, dev_tied, B, P + G)
    print(f"case full-size {name} B={B} P={P}, tied blocks", flush=True)
    gpu = helpers.gpu_generate(full, None, prompts, G, alpha, start, forced=forced, decoder=dec, fill_each_step=True)

    oracle.set_threads(helpers.oracle_threads())
    model = oracle.OracleModel(one, w1)
    def rel(a, b):
        return float(np.linalg.norm(a - b) / np.linalg.norm(b))
    worst_l = worst_h = 0.0
    for b in (0, B - 1):
        seq = model.new_seq(P + G)
        for p in range(P - 1):
            seq.first_block_kv(int(prompts[b, p]), p, 0)
        hid, _ = seq.forward_token(int(prompts[b, P - 1]), P - 1, [0], want_hidden=True)
        e = rel(gpu["hidden"][0][1, b].astype(np.float64), hid[1])
        worst_h = max(worst_h, e)
        assert e <= helpers.HIDDEN_REL_L2, f"seq {b} prompt: hidden rel L2 {e:.3e}"
        for i in range(1, G):
            blocks = [0] if keep[i] >= 1 else []
            h, lg = seq.forward_token(int(forced[b, i - 1]), P + i - 1, blocks, want_hidden=True, want_logits=True)
            got = gpu["hidden"][i][:, b].astype(np.float64)
            assert rel(got[0], h[0]) <= 1e-6                               # the embedding row
            if keep[i] >= 1:
                e = rel(got[1], h[1])
                worst_h = max(worst_h, e)
                assert e <= helpers.HIDDEN_REL_L2, f"seq {b} step {i}: hidden rel L2 {e:.3e}"
            if keep[i] <= 1:                                                # logits depend on block 0 at most
                err = float(np.abs(gpu["logits"][i][b].astype(np.float64) - lg).max())
                worst_l = max(worst_l, err)
                assert err <= helpers.LOGIT_ATOL, f"seq {b} step {i}: logits max abs err {err:.3e}"
                top2 = np.partition(lg, -2)[-2:]
                if top2[1] - top2[0] > helpers.TOKEN_MARGIN:
                    assert int(gpu["tokens"][i][b]) == oracle.argmax(lg)
    print(f"  worst logit abs err {worst_l:.3e}, worst hidden rel L2 {worst_h:.3e}", flush=True)
    # the fill of the dropped blocks copied the source block's rows (bit-exact), at full cache size
    i = 1
    pos, s, n = P + i - 1, int(drop[i]), full.L - int(keep[i])
    assert s >= 1 and torch.equal(dec.k_cache[s, B - 1, :, pos], dec.k_cache[s - 1, B - 1, :, pos])
    assert torch.equal(dec.v_cache[s + n - 1, 0, :, pos], dec.v_cache[s - 1, 0, :, pos])
    dec.close()


@pytest.mark.parametrize("V,B", [(64, 2), (1024, 1), (2050, 3), (32768, 2), (32770, 1), (65602, 2)])
@pytest.mark.parametrize("kind", ["drawn", "every logit twice", "some not numbers", "all equal", "no numbers", "the last one"])
def test_greedy_token_is_the_first_of_the_largest_logits(V, B, kind):
    # rows of less than a wave's pairs, of one and of several rounds of 32768 logits and one pair more; exact, against the returned logits
    import torch
    from paper_2503_08524_amd import binding
    s = ModelShape("argmax", L=1, d=64, H=1, H_kv=1, hd=64, F=64, V=V, dtype="f32")
    w = binding.weights_to_device(s, d3_inputs.make_weights(s, 3), "cuda:0")
    head = w["lm_head"]
    if kind == "every logit twice":
        head[V // 2:] = head[:V // 2].clone()
    elif kind == "some not numbers":
        head[::3] = float("nan")
    elif kind == "all equal":
        head.zero_()
    elif kind == "no numbers":
        head.fill_(float("nan"))
    dec = binding.Decoder(s, w, B, 8, kv_dtype="f32")
    tok, lg = torch.empty(B, dtype=torch.int32, device="cuda:0"), torch.empty(B, V, device="cuda:0")
    prompt = torch.from_numpy(d3_inputs.make_prompt(B, 3, V, seed=5)).to("cuda:0")
    dec.prefill(prompt, next_tok=tok, logits=lg)
    if kind == "the last one":                         # ... of the first sequence: a row of the head along its final hidden state
        dec.close()
        head[V - 1] = 50.0 * head[int(tok[0])]
        dec = binding.Decoder(s, w, B, 8, kv_dtype="f32")
        dec.prefill(prompt, next_tok=tok, logits=lg)
    torch.cuda.synchronize()
    x = lg.cpu().numpy()
    want = [0 if np.isnan(r).all() else int(np.nanargmax(r)) for r in x]
    assert tok.cpu().tolist() == want
    if kind == "the last one":
        assert want[0] == V - 1
    dec.close()

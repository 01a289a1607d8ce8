"""Layer stack on the GPU against the stack oracle: prompt through prefill (first token from the base
model), then greedy token steps with one encoder row and decoder rows per sequence.

Floating point decides an integer here (the greedy token).  Logits are compared to tolerance; a
token must equal the oracle's wherever the oracle's two best logits are further apart than twice the
logit tolerance, and must in any case be a logit within that margin of the oracle's best."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _build(shape, n_layers, vocab, num_blocks, seed, lora_std=0.05, kv_scales=None):
    import dataclasses
    import oracle
    from gpu_util import dev, make_layer
    from helpers import oracle_config
    from paper_2603_13281_amd import binding, synth
    wts = synth.make_stack(shape, n_layers, vocab, seed=seed, lora_std=lora_std)
    cfg = oracle_config(shape, num_blocks)
    kw = {}
    if kv_scales is not None:      # FP8 cache in every layer, one pair of static scales
        cfg = dataclasses.replace(cfg, kv_fp8=True, k_scale=kv_scales[0], v_scale=kv_scales[1])
        kw = dict(kv_fp8=True, k_scale=kv_scales[0], v_scale=kv_scales[1])
    orc = oracle.OracleStack([oracle.Oracle(cfg, b, l) for b, l in zip(wts["bases"], wts["loras"])],
                             wts["embed"], wts["final_norm"], wts["lm_head"])
    layers = [make_layer(shape, b, l, num_blocks, **kw) for b, l in zip(wts["bases"], wts["loras"])]
    stack = binding.IcarusStack(layers, dev(wts["embed"], shape.bf16), dev(wts["final_norm"], shape.bf16), dev(wts["lm_head"], shape.bf16))
    pools = [torch.zeros(layers[0].cfg.pool_shape(), dtype=layers[0].cfg.pool_dtype, device="cuda:0") for _ in layers]
    return wts, orc, stack, pools


def _check_tokens(got_tok, got_logits, want_logits, tol, what):
    scale = np.abs(want_logits).max()
    err = np.abs(got_logits - want_logits).max()
    assert err <= tol * scale, f"{what}: logits off by {err / scale:.3g} of their range (tolerance {tol})"
    for r in range(want_logits.shape[0]):
        order = np.argsort(-want_logits[r], kind="stable")
        best, second = want_logits[r, order[0]], want_logits[r, order[1]]
        assert want_logits[r, got_tok[r]] >= best - 2 * tol * scale, f"{what}: row {r} took a token that is not near the best"
        if best - second > 2 * tol * scale:
            assert got_tok[r] == order[0], f"{what}: row {r} token {got_tok[r]} != {order[0]}"


@pytest.mark.parametrize("kind", ["tiny-fp32", "llama-small-bf16", "qwen-small-bf16", "llama-small-fp8kv"])
def test_stack_prefill_then_greedy_decode(kind):
    from paper_2603_13281_amd import synth
    shape, n_layers, vocab, tol = {
        "tiny-fp32": (synth.TINY, 3, 264, 1e-4),
        "llama-small-bf16": (synth.LLAMA_SMALL, 3, 1024, 2e-2),
        "qwen-small-bf16": (synth.QWEN_SMALL, 2, 512, 2e-2),
        "llama-small-fp8kv": (synth.LLAMA_SMALL, 3, 1024, 2e-2),
    }[kind]
    kv_scales = (0.02, 0.02) if kind.endswith("fp8kv") else None
    S, steps = 3, 4
    rng = np.random.default_rng(4)
    prompt_lens = np.array([37, 5, 64], dtype=np.int32)
    Bk = shape.block_size
    max_blocks = int((prompt_lens.max() + steps + Bk) // Bk) + 1
    num_blocks = S * max_blocks + 2
    wts, orc, stack, pools = _build(shape, n_layers, vocab, num_blocks, seed=11, kv_scales=kv_scales)
    opools = orc.new_pools()
    bt = rng.permutation(num_blocks)[:S * max_blocks].reshape(S, max_blocks).astype(np.int32)
    dbt = torch.from_numpy(bt).to("cuda:0")
    tokens = rng.integers(0, vocab, size=int(prompt_lens.sum())).astype(np.int32)
    zeros = np.zeros(S, dtype=np.int32)

    # prompt: first token from the base model
    nxt, lg = stack.prefill(pools, dbt, zeros, prompt_lens, tokens, want_logits=True)
    want_lg, want_tok = orc.prefill(opools, bt, zeros, prompt_lens, tokens)
    torch.cuda.synchronize()
    _check_tokens(nxt.cpu().numpy(), lg.cpu().numpy().astype(np.float64), want_lg, tol, f"{kind} prefill")

    # greedy steps: sequence s runs 1 + m_s rows; the sequence's last row decides its next token.
    # Both sides are fed the ORACLE's token each step, so that a legitimate near-tie cannot fork them.
    row_seq = np.int32([0, 0, 1, 1, 1, 2])
    row_model = np.int32([-1, 1, -1, 0, 1, -1])
    last_row = np.array([1, 4, 5])
    ctx = prompt_lens.copy()
    cur = want_tok.astype(np.int32)
    for t in range(steps):
        seq_tok = torch.from_numpy(cur).to("cuda:0")
        seq_next = torch.empty(S, dtype=torch.int32, device="cuda:0")
        row_next, lg = stack.decode(pools, dbt, ctx, row_seq, row_model, seq_tok, seq_next=seq_next, want_logits=True)
        want_lg, want_row_tok, _ = orc.decode(opools, bt, ctx, row_seq, row_model, cur)
        torch.cuda.synchronize()
        got_rows = row_next.cpu().numpy()
        _check_tokens(got_rows, lg.cpu().numpy().astype(np.float64), want_lg, tol, f"{kind} step {t}")
        np.testing.assert_array_equal(seq_next.cpu().numpy(), got_rows[last_row])
        cur = want_row_tok[last_row].astype(np.int32)
        ctx = ctx + 1


@pytest.mark.parametrize("prompt_lens", [(20, 13), (20, 14), (1, 33), (300,)])
@pytest.mark.parametrize("n_layers", [1, 2])
def test_prompt_whose_last_layer_keeps_one_row_of_each_chunk(prompt_lens, n_layers):
    """From 32 rows more than chunks on the last layer's projections run for the chunks' last rows alone: both sides of that line, a
    chunk of one row, and a single layer (which is the first one too) against the oracle."""
    from gpu_util import pool_from_device_layout
    from paper_2603_13281_amd import synth
    shape, vocab, tol = synth.QWEN_SMALL, 512, 2e-2
    lens = np.array(prompt_lens, np.int32)
    S = len(lens)
    max_blocks = int(lens.max() + 8) // shape.block_size + 1
    num_blocks = S * max_blocks
    rng = np.random.default_rng(5)
    wts, orc, stack, pools = _build(shape, n_layers, vocab, num_blocks, seed=3)
    opools = orc.new_pools()
    bt = rng.permutation(num_blocks).reshape(S, max_blocks).astype(np.int32)
    tokens = rng.integers(0, vocab, size=int(lens.sum())).astype(np.int32)
    zeros = np.zeros(S, np.int32)
    nxt, lg = stack.prefill(pools, torch.from_numpy(bt).to("cuda:0"), zeros, lens, tokens, want_logits=True)
    want_lg, _ = orc.prefill(opools, bt, zeros, lens, tokens)
    torch.cuda.synchronize()
    _check_tokens(nxt.cpu().numpy(), lg.cpu().numpy().astype(np.float64), want_lg, tol, f"{prompt_lens}")
    for l in range(n_layers):  # every row's K and V are in the cache, those of rows that do not leave the last layer too
        got, want = pool_from_device_layout(pools[l].float().cpu().numpy(), shape.block_size, shape.head_dim), opools[l]
        assert np.linalg.norm(got - want) <= 1e-2 * np.linalg.norm(want)


@pytest.mark.parametrize("modes", [(0, 1, 0), (1, 0, 0), (0, 0, 1), (1, 0, 1, 0)], ids=lambda m: "".join(map(str, m)))
@pytest.mark.parametrize("kind", ["norms", "fp8"])
def test_prompt_through_layers_of_different_kernel_modes(kind, modes):
    """Rows enough for the projection that appends by itself; its table of angles and slots stands where the layers of mode 1 put their
    projections, so a layer may take it over from the one before it only if that one left it."""
    from gpu_util import fp8_pool_to_float, pool_from_device_layout
    from paper_2603_13281_amd import binding, synth
    print("case: kernel modes", kind, modes, flush=True)
    shape, vocab, tol = synth.QWEN_SMALL if kind == "norms" else synth.LLAMA_SMALL, 512, 2e-2
    scales = (0.02, 0.02) if kind == "fp8" else None
    lens = np.array([149, 151], np.int32)
    qd, kvd = shape.n_q_heads * 128, shape.n_kv_heads * 128
    tile = binding.gemm_choice(int(lens.sum()), shape.d_model, [qd, kvd, kvd], taken=True)
    assert tile[0] >= 128 and tile[3] == 1, tile  # several row tiles, one slice: the fused form
    S, max_blocks = len(lens), int(lens.max()) // shape.block_size + 1
    wts, orc, stack, pools = _build(shape, len(modes), vocab, S * max_blocks, seed=9, kv_scales=scales)
    opools = orc.new_pools()
    rng = np.random.default_rng(9)
    bt = rng.permutation(S * max_blocks).reshape(S, max_blocks).astype(np.int32)
    tokens = rng.integers(0, vocab, size=int(lens.sum())).astype(np.int32)
    zeros = np.zeros(S, np.int32)
    for layer, mode in zip(stack.layers, modes):
        layer.set_kernel_mode(mode)
    nxt, lg = stack.prefill(pools, torch.from_numpy(bt).to("cuda:0"), zeros, lens, tokens, want_logits=True)
    want_lg, _ = orc.prefill(opools, bt, zeros, lens, tokens)
    torch.cuda.synchronize()
    _check_tokens(nxt.cpu().numpy(), lg.cpu().numpy().astype(np.float64), want_lg, tol, f"modes {modes}")
    for l, want in enumerate(opools):
        got = fp8_pool_to_float(pools[l], *scales) if scales else pools[l].float().cpu().numpy()
        got = pool_from_device_layout(got, shape.block_size, shape.head_dim)
        # FP8: a code rounds to its neighbour, 2^-3 of its size away at most, for no more than one value in four
        assert np.linalg.norm(got - want) <= (2.0 ** -4 if scales else 1e-2) * np.linalg.norm(want), l


def test_stack_rejects_bad_arguments():
    from paper_2603_13281_amd import binding, synth
    shape = synth.TINY
    wts, orc, stack, pools = _build(shape, 2, 64, 8, seed=1)
    dbt = torch.arange(4, dtype=torch.int32, device="cuda:0").reshape(1, 4)
    with pytest.raises(binding.IcarusError) as e:       # token outside the vocabulary
        stack.prefill(pools, dbt, [0], [3], [1, 2, 64])
    assert e.value.status_name == "INVALID_ARG"
    with pytest.raises(binding.IcarusError) as e:       # context beyond the block table
        stack.prefill(pools, dbt, [0], [4 * shape.block_size + 1], np.zeros(4 * shape.block_size + 1, dtype=np.int32))
    assert e.value.status_name == "CAPACITY"
    with pytest.raises(binding.IcarusError) as e:       # two encoder rows in one sequence
        stack.decode(pools, dbt, [3], [0, 0], [-1, -1], torch.zeros(1, dtype=torch.int32, device="cuda:0"))
    assert e.value.status_name == "ROW_ORDER"


def test_stack_with_a_wide_vocabulary():
    """The LM head of a few rows against a vocabulary of more column tiles than a round of workgroups, with a ragged
    last one; prompt (2 logit rows) and one token step (5 rows)."""
    from paper_2603_13281_amd import synth
    print("case: wide vocabulary", flush=True)
    shape = synth.LLAMA_SMALL.replace(d_model=256, d_ffn=512)
    vocab, tol = 448 * 256 + 24, 2e-2
    lens = np.array([20, 7], dtype=np.int32)
    wts, orc, stack, pools = _build(shape, 1, vocab, 6, seed=13)
    opools = orc.new_pools()
    bt = np.arange(6, dtype=np.int32).reshape(2, 3)
    dbt = torch.from_numpy(bt).to("cuda:0")
    rng = np.random.default_rng(13)
    tokens = rng.integers(0, vocab, size=int(lens.sum())).astype(np.int32)
    zeros = np.zeros(2, dtype=np.int32)
    nxt, lg = stack.prefill(pools, dbt, zeros, lens, tokens, want_logits=True)
    want_lg, _ = orc.prefill(opools, bt, zeros, lens, tokens)
    torch.cuda.synchronize()
    _check_tokens(nxt.cpu().numpy(), lg.cpu().numpy().astype(np.float64), want_lg, tol, "wide vocabulary prefill")
    row_seq, row_model = np.int32([0, 0, 0, 1, 1]), np.int32([-1, 0, 2, -1, 3])
    cur = rng.integers(0, vocab, size=2).astype(np.int32)
    got, lg = stack.decode(pools, dbt, lens, row_seq, row_model, torch.from_numpy(cur).to("cuda:0"), want_logits=True)
    want_lg, _, _ = orc.decode(opools, bt, lens, row_seq, row_model, cur)
    torch.cuda.synchronize()
    _check_tokens(got.cpu().numpy(), lg.cpu().numpy().astype(np.float64), want_lg, tol, "wide vocabulary decode")

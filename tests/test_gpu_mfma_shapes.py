"""The MFMA projections at the edges of their row tiles, large prompt passes, and activations and
weights whose magnitudes lie far apart (the projections cut activations into two fp16 parts of a
row-wise scaled value and keep weights as fp16 scaled by rows), against the CPU oracle."""
import numpy as np
import pytest

import workloads as wl
from parity_util import TOL, compare_run, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_09215_amd import binding
    return binding


# input widths that are no multiple of a 64-wide chunk, task counts that end inside a tile
SHAPE = wl.TINY.shape.replace(name="bf16-edges", dtype=wl.DTYPE_BF16, n_layers=3, d_model=264, n_q_heads=7,
                              n_kv_heads=1, head_dim=128, d_ffn=1024 + 40, vocab_text=900, vocab_speech=301)


@pytest.mark.parametrize("B", [5, 16, 31, 32, 33, 48, 49, 64, 65, 96, 97, 128, 129])
def test_rows_at_the_edges_of_the_tiles(sb, B):
    """B sequences on the same schedule: B rows in every pass of the lower layers and of the heads
    (48 is the last count without LDS, 64, 96 and 128 fill a tile of two, three and four blocks of
    rows, 129 starts a second tile), up to 4 B in the flushes"""
    say(f"case {B} rows")
    weights = wl.make_weights(SHAPE, seed=11, gain_std=0.1)
    prompts = [wl.make_prompt(SHAPE, 1 + i % 3, seed=60 + i) for i in range(B)]
    sp = sb.Spark(SHAPE, wl.TINY.schedule, weights, max_batch=B, max_seq_len=64, kv_page_tokens=16)
    compare_run(sp, SHAPE, wl.TINY.schedule, weights, prompts, [0] * B, 7, label=f"{B} rows")
    sp.close()


@pytest.mark.parametrize("n,page,group,shared", [(34, 64, 7, 1), (65, 16, 7, 1), (66, 64, 2, 1), (130, 16, 16, 1), (386, 64, 7, 1),
                                                 (1025, 64, 16, 1), (1102, 16, 7, 1), (130, 16, 7, 0), (600, 64, 16, 0),
                                                 (1102, 16, 2, 0)])
def test_prompt_lengths(sb, n, page, group, shared):
    """shared: the rows of passes of 64 and more share K and V, otherwise as the library chooses.
    Prompts of one pass and of two (1024 rows is the largest pass), ragged last tiles of rows and of
    tokens, pages smaller than an attention tile, 16, 7 and 2 query heads per KV head: cache entries of
    every position and the steps behind the prompt"""
    say(f"case prompt of {n}, pages of {page}, {group} heads, shared {shared}")
    shape = SHAPE.replace(n_q_heads=2 * group, n_kv_heads=2)
    weights = wl.make_weights(shape, seed=12, gain_std=0.1)
    sp = sb.Spark(shape, wl.TINY.schedule, weights, max_batch=1, max_seq_len=n + 64, kv_page_tokens=page)
    if shared:
        sp.tune("attn_prompt_min_rows", 64)
    compare_run(sp, shape, wl.TINY.schedule, weights, [wl.make_prompt(shape, n, seed=61)], [0], 3, check_kv_every=2,
                label=f"prompt {n}", kv_all_positions=n < 400)
    sp.close()


# inputs long enough that k is cut
LONG_K = SHAPE.replace(name="bf16-long-k", d_model=1032, n_q_heads=8, n_kv_heads=2, d_ffn=1304)


@pytest.mark.parametrize("B,tune", [(6, {}), (6, dict(direct_whole_k=64)), (19, dict(direct_whole_k=64)), (19, dict(direct_whole_k=8192)),
                                    (40, dict(direct_whole_k=-1)), (6, dict(direct_max_rows=0)),
                                    (30, dict(direct_max_rows=16)), (36, {}), (36, dict(tiled_row_blocks=2)),
                                    (52, {}), (70, dict(tiled_row_blocks=2)), (52, dict(fuse_norm=0)), (40, dict(direct_max_rows=32)),
                                    (36, dict(fuse_norm=0)), (6, dict(fuse_norm=0)), (12, dict(mfma_tiled=0)),
                                    (36, dict(mfma_tiled=0)), (36, dict(mfma_tiled=0, fuse_norm=0))])
def test_projection_kernels_by_their_switches(sb, B, tune):
    """the kernels that the switches lead to, k cut and whole, on the same rows: without LDS and with it
    for at most 48 rows, row tiles of two blocks, norms as launches, the caller's weights"""
    say(f"case {B} rows, {tune}")
    weights = wl.make_weights(LONG_K, seed=15, gain_std=0.1)
    prompts = [wl.make_prompt(LONG_K, 1 + i % 3, seed=60 + i) for i in range(B)]
    sp = sb.Spark(LONG_K, wl.TINY.schedule, weights, max_batch=B, max_seq_len=64, kv_page_tokens=16)
    for name, value in tune.items():
        sp.tune(name, value)
    compare_run(sp, LONG_K, wl.TINY.schedule, weights, prompts, [0] * B, 6, label=f"{B} rows {tune}")
    sp.close()


@pytest.mark.parametrize("B", [3, 4, 8, 9, 16, 17, 32, 33, 47, 48])
def test_rows_at_the_edges_of_the_direct_kernels(sb, filled_scratch, B):
    """one operand of 16 activation rows to three, one tile a workgroup (up to 8 rows) or a round of CUs;
    inputs of 1024, 1032 and 1304, two of them no multiples of a chunk (what lies behind their last row of
    k is NaN), cut in two from 9 rows on; three and four rows: on the vector kernels, flushes on these"""
    say(f"case direct kernels, {B} rows")
    weights = wl.make_weights(LONG_K, seed=18, gain_std=0.1)
    prompts = [wl.make_prompt(LONG_K, 1 + i % 3, seed=80 + i) for i in range(B)]
    sp = sb.Spark(LONG_K, wl.TINY.schedule, weights, max_batch=B, max_seq_len=64, kv_page_tokens=16)
    compare_run(sp, LONG_K, wl.TINY.schedule, weights, prompts, [0] * B, 6, label=f"{B} rows")
    sp.close()


def test_flush_of_more_rows_than_a_pass_takes(sb):
    """256 sequences with fifteen pending positions each complete them on the same step: 4096 rows, which
    go through the upper layers in two pieces (3072 at this width); the sequences' logits are those that
    a few of them have alone"""
    import torch
    say("case flush of 4096 rows")
    shape = SHAPE.replace(n_layers=2, d_model=4096, n_q_heads=2, n_kv_heads=1, d_ffn=72, vocab_text=0, vocab_speech=300)
    sched = wl.TINY.schedule.replace(exit_layer=1, period_k=16, phase=15, n_text=0, n_speech=1, scope=wl.SCOPE_STREAM)
    weights = wl.make_weights(shape, seed=16, gain_std=0.1)
    rng = np.random.default_rng(9)
    first, forced = rng.integers(0, 300, 256), rng.integers(0, 300, (16, 256))

    def run(which):
        sp = sb.Spark(shape, sched, weights, max_batch=len(which), max_seq_len=32, kv_page_tokens=16)
        ids = [sp.seq_open(0) for _ in which]
        for i, b in zip(ids, which):
            sp.prefill(i, [int(first[b])])
        _, depth = sp.decode(16, ids, forced[:, which])
        assert np.all(depth[:15] == 1) and np.all(depth[15] == 2)
        out = np.stack([sp.get_logits(i)[0] for i in ids])
        assert sp.get_stats(ids[0])["flush_hist"] == {16: 1}
        sp.close()
        return out

    some = [0, 1, 100, 191, 192, 193, 254, 255]   # 191 and 192: the rows around the cut
    assert np.max(np.abs(run(list(range(256)))[some] - run(some))) <= TOL[wl.DTYPE_BF16]
    torch.cuda.empty_cache()


def test_prompt_without_the_large_buffers(sb, monkeypatch):
    """a scratch area one byte short of the buffers of 1024-row passes: the copy of the weights and
    passes in the buffers that every context has"""
    say("case prompt without the large buffers")
    lib = sb.load_library()
    init = lib.spark_init
    weights = wl.make_weights(SHAPE, seed=12, gain_std=0.1)
    monkeypatch.setattr(lib, "spark_init", lambda c, w, kv, kvb, sc, scb, st, out: init(c, w, kv, kvb, sc, scb - 1, st, out))
    sp = sb.Spark(SHAPE, wl.TINY.schedule, weights, max_batch=1, max_seq_len=660, kv_page_tokens=64)
    compare_run(sp, SHAPE, wl.TINY.schedule, weights, [wl.make_prompt(SHAPE, 600, seed=61)], [0], 3, check_kv_every=2,
                label="prompt without the large buffers", kv_all_positions=True)
    sp.close()


def test_prompt_rows_can_be_set_and_unset(sb):
    """"prefill_rows": passes of a set size, up to that of the large buffers, and back to the size that
    a new context chooses"""
    say("case prompt rows set and unset")
    weights = wl.make_weights(SHAPE, seed=12, gain_std=0.1)
    prompt = wl.make_prompt(SHAPE, 600, seed=61)

    def entries(*values):
        sp = sb.Spark(SHAPE, wl.TINY.schedule, weights, max_batch=1, max_seq_len=640, kv_page_tokens=64)
        for v in values:
            sp.tune("prefill_rows", v)
        sid = sp.seq_open(0)
        sp.prefill(sid, prompt)
        out = np.stack([np.concatenate(sp.get_kv(sid, SHAPE.n_layers - 1, p)) for p in range(599)])
        sp.close()
        return out

    default = entries()
    assert np.array_equal(default, entries(128, 0))       # unset: the same passes, bit by bit
    assert not np.array_equal(default, entries(32))       # other passes: other k ranges, other roundings
    assert np.array_equal(default, entries(640))          # one pass of 599 rows either way
    for rows in (32, 256, 320, 1024, 5000):
        assert np.max(np.abs(default - entries(rows))) <= TOL[wl.DTYPE_BF16] + 2.0 ** -7 * np.abs(default).max()


@pytest.mark.parametrize("n,at,page", [(130, 70, 64), (130, 127, 16), (200, 3, 64), (1030, 1020, 64)])
def test_a_nan_stays_behind_its_position(sb, n, at, page):
    """a prompt with a token whose embedding is NaN: cache entries of the positions before it are
    those of the same prompt without it, bit by bit, and from it on none is finite in the upper layers"""
    say(f"case NaN at {at} of {n}")
    shape = SHAPE.replace(n_q_heads=14, n_kv_heads=2)
    weights = wl.make_weights(shape, seed=12, gain_std=0.1)
    bad = shape.vocab - 1
    weights["embed"][bad] = wl.f32_to_bf16_bits(np.full(shape.d_model, np.nan, dtype=np.float32))
    prompt = wl.make_prompt(shape, n, seed=61) % bad
    marked = prompt.copy()
    marked[at] = bad
    sp = sb.Spark(shape, wl.TINY.schedule, weights, max_batch=2, max_seq_len=n + 64, kv_page_tokens=page)
    sp.tune("attn_prompt_min_rows", 64)
    a, b = sp.seq_open(0), sp.seq_open(0)
    sp.prefill(a, prompt)
    sp.prefill(b, marked)
    top = shape.n_layers - 1
    for pos in range(n - 1):
        if pos < at:
            for layer in (1, top):
                for want, got in zip(sp.get_kv(a, layer, pos), sp.get_kv(b, layer, pos)):
                    assert np.array_equal(want, got), (layer, pos)
        else:
            assert all(np.all(np.isnan(x)) for x in sp.get_kv(b, top, pos)), pos
    sp.close()


@pytest.fixture
def filled_scratch():
    """torch.empty filled with 0xff bytes: what the scratch area holds that nobody has written"""
    import torch
    before = torch.are_deterministic_algorithms_enabled(), torch.utils.deterministic.fill_uninitialized_memory
    torch.use_deterministic_algorithms(True)
    torch.utils.deterministic.fill_uninitialized_memory = True
    assert int(torch.empty(64, dtype=torch.uint8, device="cuda:0").min()) == 255
    yield
    torch.use_deterministic_algorithms(before[0])
    torch.utils.deterministic.fill_uninitialized_memory = before[1]


@pytest.mark.parametrize("n,shape_kw,tune", [
    # more rows than the slices' partial results hold at a time, one to five in the second turn
    (258, dict(n_q_heads=16, head_dim=64), {}), (260, dict(n_q_heads=14, n_kv_heads=2, head_dim=64), {}),
    (261, dict(n_q_heads=16, head_dim=64), {}), (262, dict(n_q_heads=16, head_dim=64), {}),
    (259, dict(n_q_heads=16), dict(attn_prompt_min_rows=2000)),
    (560, dict(n_q_heads=16), dict(attn_prompt_min_rows=2000)),
])
def test_prompt_attention_in_turns(sb, filled_scratch, n, shape_kw, tune):
    """passes whose rows do not share K and V and are attended in turns: every row's list of
    magnitudes, as long as the output projection reads it, has been written"""
    say(f"case prompt of {n} in turns, {shape_kw} {tune}")
    shape = SHAPE.replace(**shape_kw)
    weights = wl.make_weights(shape, seed=12, gain_std=0.1)
    sp = sb.Spark(shape, wl.TINY.schedule, weights, max_batch=1, max_seq_len=n + 64, kv_page_tokens=64)
    for name, value in tune.items():
        sp.tune(name, value)
    compare_run(sp, shape, wl.TINY.schedule, weights, [wl.make_prompt(shape, n, seed=61)], [0], 3, check_kv_every=2,
                label=f"prompt {n} in turns", kv_all_positions=True)
    sp.close()


@pytest.mark.parametrize("pieces,long", [(0, 62), (0, 126), (0, 700), (8, 62), (8, 510), (8, 700), (2, 126)])
def test_attention_workgroups(sb, pieces, long):
    """contexts that grow over the edge of a 64-token piece, of a pair of pieces and of a workgroup's
    pieces, with two teams of waves per workgroup (pieces 8, and 0: as the library chooses for so few
    rows) and with one (2): the second team with no piece at all, with fewer than the first, as many"""
    say(f"case attention workgroups, {pieces} pieces, {long} tokens")
    shape = SHAPE.replace(n_q_heads=32, n_kv_heads=2)
    weights = wl.make_weights(shape, seed=14, gain_std=0.1)
    sp = sb.Spark(shape, wl.TINY.schedule, weights, max_batch=3, max_seq_len=long + 64, kv_page_tokens=16)
    sp.tune("attn_pieces", pieces)
    prompts = [wl.make_prompt(shape, n, seed=90 + n) for n in (long, long // 2, 3)]
    compare_run(sp, shape, wl.TINY.schedule, weights, prompts, [0, 1, 2], 7, check_kv_every=2,
                label=f"{pieces} pieces, {long} tokens")
    sp.close()


@pytest.mark.parametrize("pieces,page", [(0, 64), (1, 64), (2, 64), (2, 16)])
def test_attention_waves_without_tokens(sb, pieces, page):
    """contexts that grow over the edges of a wave's 16 tokens: pieces of which one to four waves have tokens,
    in one slice and in the last of several"""
    say(f"case attention waves, {pieces} pieces, pages of {page}")
    weights = wl.make_weights(SHAPE, seed=14, gain_std=0.1)
    sp = sb.Spark(SHAPE, wl.TINY.schedule, weights, max_batch=4, max_seq_len=256, kv_page_tokens=page)
    sp.tune("attn_pieces", pieces)
    prompts = [wl.make_prompt(SHAPE, n, seed=90 + n) for n in (12, 29, 45, 140)]
    compare_run(sp, SHAPE, wl.TINY.schedule, weights, prompts, [0, 1, 2, 0], 8, check_kv_every=4, label=f"{pieces} pieces, pages of {page}")
    sp.close()


@pytest.mark.parametrize("B", [6, 40, 70])
def test_magnitudes_far_apart(sb, B):
    """(The kernel without LDS with one operand of rows and with three, and the one with it.)  Gains of 2^-30 and 2^30 with weights that undo them, and MLP activations spread over a factor
    of 1024 within a row, undone by the columns of the down projection: powers of two, so that the
    model is the same one.  What the two fp16 parts leave out is 2^-23 of an element or 2^-40 of its
    row's largest, 2^-30 of the smallest elements here, so the tolerance is that of any bf16 model."""
    say(f"case magnitudes, {B} rows")
    weights = wl.make_weights(SHAPE, seed=13, gain_std=0.1)

    def times(bits, power):   # exact: no weight comes near the ends of the exponent range
        return wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(bits) * np.exp2(power).astype(np.float32))

    for gain, power, users in (("attn_norm", -30, ("wq", "wk", "wv")), ("mlp_norm", 30, ("wg", "wu")),
                               ("final_norm", -20, ("lm_head",))):
        weights[gain] = (weights[gain] * np.float32(2.0 ** power)).astype(np.float32)
        for u in users:
            weights[u] = times(weights[u], np.float32(-power))
    spread = np.random.Generator(np.random.Philox(5)).integers(-5, 6, size=SHAPE.d_ffn).astype(np.float32)
    weights["wu"] = times(weights["wu"], spread[None, :, None])
    weights["wd"] = times(weights["wd"], -spread[None, None, :])
    prompts = [wl.make_prompt(SHAPE, 3 + 7 * (i % 9), seed=80 + i) for i in range(B)]
    sp = sb.Spark(SHAPE, wl.TINY.schedule, weights, max_batch=B, max_seq_len=128, kv_page_tokens=16)
    res = compare_run(sp, SHAPE, wl.TINY.schedule, weights, prompts, [0] * B, 7, label=f"magnitudes, {B} rows")
    assert res["worst"] <= TOL[wl.DTYPE_BF16]
    sp.close()


@pytest.mark.parametrize("B,flushes", [(1, True), (2, False), (3, False), (4, False)])
def test_large_hidden_states_of_a_few_rows(sb, B, flushes):
    """hidden states 2^26 times as large as usual (a row's sum of squares around 1e15): up to four rows, also
    those of one sequence's flush, are normalised with sums in floating point, which have no upper end near there.
    The norms take the factor out again, so the tolerance is that of any bf16 model."""
    say(f"case large hidden states, {B} sequences")
    weights = wl.make_weights(SHAPE, seed=19, gain_std=0.1)
    for name in ("embed", "wo", "wd"):   # exact: powers of two
        weights[name] = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(weights[name]) * np.float32(2.0 ** 26))
    sched = wl.TINY.schedule if flushes else wl.TINY.schedule.replace(period_k=1, phase=0)
    prompts = [wl.make_prompt(SHAPE, 1 + i, seed=70 + i) for i in range(B)]
    sp = sb.Spark(SHAPE, sched, weights, max_batch=B, max_seq_len=64, kv_page_tokens=16)
    compare_run(sp, SHAPE, sched, weights, prompts, [0] * B, 7, label=f"large hidden states, {B} sequences")
    sp.close()

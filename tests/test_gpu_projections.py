"""Single projections of the MFMA path against 64 bits, with nothing behind them that would round:
models whose other matrices are zero, so that the logits are one product (the heads) or one MLP, of
fp32 activations with all their bits.  A run through many layers of a bf16 cache cannot tell parts of
activations that add up to 16 bits from parts that add up to 23: the cache rounds to 8.

Bounds (largest relative error of a row, 2-norm, without the factor that the norm's own rounding
gives the whole row).  One rounding to 32 bits leaves 0.22 * 2^-23 of the value on average (root mean
square): 2.6e-8.  Activations: two roundings in the norm, up to 2^-23 of an element (2^-24 on average)
by the two fp16 parts: 8e-8.  A sum of n MFMAs: each rounds a running sum that is half of the result's
size on average (square), sqrt(n / 2) * 2.6e-8, with n = k / 8; in segments of 80 whose sums are added,
sqrt(40) * 2.6e-8 whatever the segments' number: 1.7e-7.  The heads: 1.9e-7 in all; bound 3e-7.
Gate/up, without segments at k = 3584: 3.9e-7, times sqrt(2) for the product of the two; down 1.7e-7;
5.8e-7 in all; bound 9e-7.  (Parts that add up to 16 bits, 2^-17, leave 4e-6; one unbroken sum of the heads 5.4e-7.)"""
import numpy as np
import pytest

import workloads as wl
from parity_util import say

pytestmark = pytest.mark.gpu

D, FFN, VOCAB = 3584, 8264, 2305   # 8192 and more MLP activations: 64 tasks a wave; a down projection with its k cut


@pytest.fixture(scope="module")
def sb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_09215_amd import binding
    return binding


def model(shape, mlp):
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(21)

    def normal(*size, std=0.02):
        return (torch.randn(size, generator=gen, device="cuda:0") * std).bfloat16()

    W = {}
    for name, size in wl.tensor_shapes(shape).items():
        if name in wl.GAIN_TENSORS:
            W[name] = 1.0 + 0.1 * torch.randn(size, generator=gen, device="cuda:0")
        elif name in wl.FP32_TENSORS:
            W[name] = torch.zeros(size, device="cuda:0")
        elif name in ("wo", "wd", "lens_a"):
            W[name] = torch.zeros(size, device="cuda:0").bfloat16()
        else:
            W[name] = normal(*size, std=0.05 if mlp and name == "embed" else 1.0 if name == "embed" else 0.02)
    if mlp:   # the second layer and the head leave the first layer's result as it is
        W["wd"][0] = normal(*W["wd"][0].shape)
        W["lm_head"] = torch.eye(D, device="cuda:0").bfloat16()
        W["final_norm"] = torch.ones(D, device="cuda:0")
    W["lens_head"] = W["lm_head"]
    return W


def norm64(x, gain, eps):
    import torch
    x = x.double()
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def row_errors(got, want):
    import torch
    got = torch.as_tensor(np.stack(got)).to(want.device).double()
    factor = (got * want).sum(-1, keepdim=True) / (want * want).sum(-1, keepdim=True)
    assert float((factor - 1).abs().max()) < 1e-6
    return ((got - factor * want).norm(dim=-1) / want.norm(dim=-1)).cpu().numpy()


def first_step(spark, tokens, full=None):
    """one step of sequences that hold one token each; full: those that run full depth at once"""
    ids = [spark.seq_open(0) for _ in tokens]
    for i, t in zip(ids, tokens):
        spark.prefill(i, [int(t)])
    for b in full if full is not None else []:
        spark.seq_set_phase(ids[b], 0)
    _, depth = spark.step(ids)
    return ids, depth


@pytest.mark.parametrize("rows,spread", [(5, 0), (32, 0), (33, 0), (48, 0), (49, 0), (64, 0), (96, 0), (128, 0), (129, 0), (7, 60), (70, 60)])
def test_head_against_64_bits(sb, rows, spread):
    """spread: the vocabulary's rows times powers of two between 2^-spread and 2^spread (their logits
    are compared without them): neighbouring rows share tiles, and nothing else"""
    import torch
    say(f"case head alone, {rows} rows, spread {spread}")
    shape = wl.TINY.shape.replace(name="head", dtype=wl.DTYPE_BF16, n_layers=1, d_model=D, n_q_heads=2, n_kv_heads=1,
                                  head_dim=128, d_ffn=64, vocab_text=VOCAB, vocab_speech=0)
    sched = wl.TINY.schedule.replace(exit_layer=1, period_k=1, phase=0, n_text=1, n_speech=0)
    W = model(shape, False)
    power = torch.as_tensor(np.random.default_rng(3).integers(-spread, spread + 1, VOCAB), device="cuda:0")
    W["lm_head"] = torch.ldexp(W["lm_head"].float(), power[:, None]).bfloat16()
    sp = sb.Spark(shape, sched, W, max_batch=rows, max_seq_len=16, kv_page_tokens=16)
    tokens = np.random.default_rng(rows).integers(0, VOCAB, rows)
    ids, _ = first_step(sp, tokens)
    x = norm64(W["embed"][torch.as_tensor(tokens, device="cuda:0")], W["final_norm"], shape.rms_eps)
    unit = torch.ldexp(torch.ones(VOCAB, device="cuda:0", dtype=torch.float64), -power)
    err = row_errors([sp.get_logits(i)[0] * unit.cpu().numpy() for i in ids], x @ W["lm_head"].double().T * unit)
    say(f"  head, {rows} rows: mean {err.mean():.3g}, largest {err.max():.3g}")
    assert err.max() <= 3e-7
    sp.close()


@pytest.mark.parametrize("rows,power,ffn", [(6, 0, FFN), (32, 0, FFN), (40, 0, FFN), (96, 0, FFN), (150, 0, FFN), (6, 50, FFN),
                                           (40, 50, FFN), (40, -50, FFN), (6, 0, 20488), (40, 0, 20480),
                                           (70, 50, FFN), (70, -50, FFN), (70, 0, 20480), (224, 0, 11272)])
def test_mlp_against_64_bits(sb, rows, power, ffn):
    """power: the up projection times 2^-power, which the down projection undoes; gate and up share
    tiles.  20480 is the longest input whose copy is written from registers.  Up to 48 rows run without LDS; 224
    with 11272 activations take lower tiles alone (180 of 256 tasks and 64 rows)."""
    import torch
    say(f"case MLP alone, {rows} rows, power {power}")
    shape = wl.TINY.shape.replace(name="mlp", dtype=wl.DTYPE_BF16, n_layers=2, d_model=D, n_q_heads=2, n_kv_heads=1,
                                  head_dim=128, d_ffn=ffn, vocab_text=0, vocab_speech=D)
    sched = wl.TINY.schedule.replace(exit_layer=1, period_k=2, phase=1, n_text=0, n_speech=1, scope=wl.SCOPE_STREAM)
    W = model(shape, True)
    W["wu"], W["wd"] = W["wu"] * 2.0 ** -power, W["wd"] * 2.0 ** power
    sp = sb.Spark(shape, sched, W, max_batch=rows, max_seq_len=16, kv_page_tokens=16)
    tokens = np.random.default_rng(rows).integers(0, D, rows)
    # four rows run full depth: their head is the vector kernel, in fp32, and shows the hidden state
    seen = sorted({0, rows // 3, 2 * rows // 3, rows - 1})
    ids, depth = first_step(sp, tokens, seen)
    assert list(np.flatnonzero(depth == 2)) == seen
    h = W["embed"][torch.as_tensor(tokens[seen], device="cuda:0")].double()
    n = norm64(h, W["mlp_norm"][0], shape.rms_eps)
    act = torch.nn.functional.silu(n @ W["wg"][0].double().T) * (n @ W["wu"][0].double().T)
    want = norm64(h + act @ W["wd"][0].double().T, W["final_norm"], shape.rms_eps)
    err = row_errors([sp.get_logits(ids[b])[0] for b in seen], want)
    say(f"  MLP, {rows} rows: mean {err.mean():.3g}, largest {err.max():.3g}")
    assert err.max() <= 9e-7
    sp.close()


@pytest.mark.parametrize("rows", [1, 2, 3, 4])
def test_mlp_of_a_few_rows_keeps_32_bits(sb, rows):
    """MLP activations between 2^-25 and 2^25 of their usual size within a row, undone by the columns of the down
    projection: up to four rows are multiplied in 32 bits with the caller's weights, so the sums are those of
    the plain model, bit for bit but for their order, and the bound is the plain model's.  (Two fp16 parts of
    a value scaled with its row would leave out all that lies 2^-39 below the row's largest.)"""
    import torch
    say(f"case MLP alone, activations far apart, {rows} rows")
    shape = wl.TINY.shape.replace(name="mlp", dtype=wl.DTYPE_BF16, n_layers=2, d_model=D, n_q_heads=2, n_kv_heads=1,
                                  head_dim=128, d_ffn=FFN, vocab_text=0, vocab_speech=D)
    sched = wl.TINY.schedule.replace(exit_layer=1, period_k=2, phase=1, n_text=0, n_speech=1, scope=wl.SCOPE_STREAM)
    W = model(shape, True)
    power = torch.as_tensor(np.random.default_rng(4).integers(-25, 26, FFN), device="cuda:0")
    W["wu"][0] = torch.ldexp(W["wu"][0].float(), power[:, None]).bfloat16()
    W["wd"][0] = torch.ldexp(W["wd"][0].float(), -power[None, :]).bfloat16()
    sp = sb.Spark(shape, sched, W, max_batch=rows, max_seq_len=16, kv_page_tokens=16)
    tokens = np.random.default_rng(rows).integers(0, D, rows)
    ids, depth = first_step(sp, tokens, range(rows))
    assert np.all(depth == 2)
    h = W["embed"][torch.as_tensor(tokens, device="cuda:0")].double()
    n = norm64(h, W["mlp_norm"][0], shape.rms_eps)
    act = torch.nn.functional.silu(n @ W["wg"][0].double().T) * (n @ W["wu"][0].double().T)
    want = norm64(h + act @ W["wd"][0].double().T, W["final_norm"], shape.rms_eps)
    err = row_errors([sp.get_logits(i)[0] for i in ids], want)
    say(f"  MLP, far apart, {rows} rows: mean {err.mean():.3g}, largest {err.max():.3g}")
    assert err.max() <= 9e-7
    sp.close()


@pytest.mark.parametrize("rows,ffn", [(1023, 8264), (700, 8264), (340, 8264), (990, 10248)])
def test_prompt_mlp_with_whole_and_cut_tiles(sb, rows, ffn):
    """gate/up of a large prompt pass: more tiles of 256 tasks x 96 rows than CUs, so that some end in the
    projection and the others in the finishing launch (33 x 11 tiles, 256 whole; 33 x 8, 256 whole), both
    of which write the rows' lists of magnitudes for the down projection; and whole tiles of two heights in one
    launch (198 of 64 rows; 247 of 96 and 265 of 64 rows).  (tests/test_partial_sums.py checks that these are the
    covers.)  Seen in the second layer's
    value entries, which are rounded to bf16: within 2^-8 of themselves and 1e-4 of a row's typical one."""
    import torch
    say(f"case MLP of a prompt of {rows}, {ffn} activations")
    d, V = 1032, 900
    shape = wl.TINY.shape.replace(name="prompt-mlp", dtype=wl.DTYPE_BF16, n_layers=2, d_model=d, n_q_heads=2, n_kv_heads=1,
                                  head_dim=128, d_ffn=ffn, vocab_text=V, vocab_speech=0)
    sched = wl.TINY.schedule.replace(exit_layer=1, period_k=1, phase=0, n_text=1, n_speech=0)
    W = model(shape, False)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    W["wd"][0] = (torch.randn(d, ffn, generator=gen, device="cuda:0") * 0.05).bfloat16()
    spread = torch.randint(-8, 9, (ffn,), generator=gen, device="cuda:0")
    W["wu"][0] = torch.ldexp(W["wu"][0].float(), spread[:, None]).bfloat16()   # activations far apart: the lists matter
    W["wd"][0] = torch.ldexp(W["wd"][0].float(), -spread[None, :]).bfloat16()
    sp = sb.Spark(shape, sched, W, max_batch=1, max_seq_len=rows + 64, kv_page_tokens=64)
    prompt = wl.make_prompt(shape, rows + 1, seed=7)
    sid = sp.seq_open(0)
    sp.prefill(sid, prompt)
    h = W["embed"][torch.as_tensor(prompt[:rows], device="cuda:0").long()].double()
    n = norm64(h, W["mlp_norm"][0], shape.rms_eps)
    act = torch.nn.functional.silu(n @ W["wg"][0].double().T) * (n @ W["wu"][0].double().T)
    v = norm64(h + act @ W["wd"][0].double().T, W["attn_norm"][1], shape.rms_eps) @ W["wv"][1].double().T
    want = v.cpu().numpy()
    typical = np.sqrt((want ** 2).mean(axis=1))
    for pos in range(0, rows, 3):
        _, got = sp.get_kv(sid, 1, pos)
        assert np.all(np.abs(got - want[pos]) <= 2.0 ** -8 * np.abs(want[pos]) + 1e-4 * typical[pos]), pos
    sp.close()

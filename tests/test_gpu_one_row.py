"""The layers of a pass of one row in one launch (one_row.h): the shapes and contexts at which its phases can go wrong,
against the oracle, and against the same steps as a launch per operation."""
from contextlib import closing

import numpy as np
import pytest

import workloads as wl
from parity_util import compare_run, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_09215_amd import binding
    binding.load_library()
    return binding


def _last_error(sp):
    return sp.lib.spark_last_error(sp.handle).decode()


def _shape(name, **over):
    return wl.TINY.shape.replace(name=name, dtype=wl.DTYPE_BF16, n_layers=4, head_dim=128, **over)


# the narrowest model (a pair of every projection for each of the 256 workgroups) and one query head per key head; widths
# that are no multiple of a unit's 512 elements nor of the workgroups, seven query heads; 16 query heads; rows of two widths
SHAPES = [
    ("narrow", dict(d_model=512, n_q_heads=2, n_kv_heads=2, d_ffn=768), 16),
    ("ragged", dict(d_model=776, n_q_heads=7, n_kv_heads=1, d_ffn=1400), 16),
    ("sixteen", dict(d_model=1024, n_q_heads=16, n_kv_heads=1, d_ffn=776), 64),
    ("wide", dict(d_model=520, n_q_heads=16, n_kv_heads=4, d_ffn=2056), 48),
]


# prompts of 1, 31 .. 33 and 62 tokens: a context of the step's own token alone, slices that fill up during the run
@pytest.mark.parametrize("name,over,page", SHAPES, ids=[s[0] for s in SHAPES])
def test_shapes(sb, name, over, page):
    w = wl.TINY
    shape = _shape(name, **over)
    weights = wl.make_weights(shape, seed=4, gain_std=0.1)
    for n in (1, 31, 62):
        say(f"one row, {name}, {n}")
        with closing(sb.Spark(shape, w.schedule, weights, max_batch=1, max_seq_len=192, kv_page_tokens=page)) as sp:
            sp.tune("one_row", 2)
            compare_run(sp, shape, w.schedule, weights, [wl.make_prompt(shape, n, seed=60)], [n % 6], 14, chunk=5, check_kv_every=7,
                        label=f"one row {name} {n}")


def _decode(sb, shape, sched, weights, prompt, steps, on, between, max_seq_len=2176):
    """forced steps of one sequence; after a few of them `between` other sequences take steps (wide passes, which leave
    other things in the area of the hand-overs)"""
    with closing(sb.Spark(shape, sched, weights, max_batch=12 if between else 1, max_seq_len=max_seq_len, kv_page_tokens=64)) as sp:
        sp.tune("one_row", on)
        sid = sp.seq_open(0)
        sp.prefill(sid, prompt)
        forced = np.arange(steps, dtype=np.int32)[:, None] % shape.vocab
        logits = []
        for at in range(0, steps, 5):
            sp.decode(min(5, steps - at), [sid], forced[at:at + 5])
            logits.append(sp.get_logits(sid)[0])
            if between:
                ids = [sp.seq_open(b) for b in range(between)]
                for b, s in enumerate(ids):
                    sp.prefill(s, wl.make_prompt(shape, 20 + b, seed=b))
                sp.decode(3, ids)
                for s in ids:
                    sp.seq_close(s)
        kv = np.concatenate(sp.get_kv(sid, 0, len(prompt) + steps - 2))
    return np.stack(logits).astype(np.float64), kv


def _same(a, ka, b, kb):
    # another order of the 32-bit sums; a cache entry may round to the neighbouring 16-bit value (2^-8 of it), which
    # moves the outputs of the layers above by far less than that
    assert np.linalg.norm(a - b) <= 2.0 ** -8 * np.linalg.norm(a)
    assert np.all(np.abs(ka - kb) <= 2.0 ** -7 * np.abs(ka) + 1e-3 * np.abs(ka).max())


# eight key heads: up to 1024 positions the slices have 32 tokens, up to 2048 64, and beyond that the steps are launches per
# operation; the second row of each pair crosses the line during the run
@pytest.mark.parametrize("n,between", [(1000, 0), (1020, 0), (2030, 0), (2045, 0), (90, 11)])
def test_contexts_and_other_passes(sb, n, between):
    shape = _shape("contexts", d_model=1024, n_q_heads=16, n_kv_heads=8, d_ffn=1536)
    weights = wl.make_weights(shape, seed=4, gain_std=0.1)
    prompt = wl.make_prompt(shape, n, seed=61)
    a, ka = _decode(sb, shape, wl.TINY.schedule, weights, prompt, 15, 0, between)
    b, kb = _decode(sb, shape, wl.TINY.schedule, weights, prompt, 15, 2, between)
    _same(a, ka, b, kb)


# a KV head's query heads are dealt to four workgroups, to two or to one as the slices become more, 16, 8 or 4 (7: 4 and 3, or 2
# and 1) to a workgroup; each run crosses a line: 32-token slices 33, 65, 129 of one KV head, 33, 65 of two, then 64-token slices
@pytest.mark.parametrize("heads,kv_heads,n", [(16, 1, 2044), (16, 1, 4092), (16, 1, 8188), (16, 2, 1020), (16, 2, 2044), (16, 2, 4092),
                                              (7, 1, 2044), (7, 1, 4092), (32, 2, 1020), (32, 2, 2044)])
def test_query_heads_of_a_workgroup(sb, heads, kv_heads, n):
    shape = _shape("heads", d_model=512, n_q_heads=heads, n_kv_heads=kv_heads, d_ffn=768)
    weights = wl.make_weights(shape, seed=4, gain_std=0.1)
    say(f"one row, {heads} heads of {kv_heads}, {n} tokens")
    prompt = wl.make_prompt(shape, n, seed=61)
    a, ka = _decode(sb, shape, wl.TINY.schedule, weights, prompt, 10, 0, 0, n + 64)
    b, kb = _decode(sb, shape, wl.TINY.schedule, weights, prompt, 10, 2, 0, n + 64)
    _same(a, ka, b, kb)


# cycle offsets, and which of the sequences then sometimes run full depth alone and with nothing pending
@pytest.mark.parametrize("offsets,which", [((0, 1), {0}), ((1, 0), {1}), ((2, 0), {0, 1}), ((5, 3, 4), {0, 1})])
def test_layers_above_the_exit_alone(sb, offsets, which):
    """several rows below the exit layer and one above it: the one launch takes the upper layers of a row that others have left"""
    w = wl.TINY
    shape = _shape("upper", d_model=1024, n_q_heads=16, n_kv_heads=8, d_ffn=1536)
    weights = wl.make_weights(shape, seed=4, gain_std=0.1)
    steps = 18
    rows = np.zeros((len(offsets), steps), dtype=int)   # above the exit layer
    for b, off in enumerate(offsets):
        pending = 0
        for g, depth in enumerate(sb.schedule_preview(shape, w.schedule, steps, off)[0]):
            full = depth == shape.n_layers
            rows[b, g] = pending + 1 if full else 0
            pending = 0 if full else pending + 1
    alone = rows.sum(0) == 1
    assert alone.sum() >= 3 and set(rows[:, alone].argmax(0)) == which
    say(f"one row above the exit layer, offsets {offsets}: {int(alone.sum())} steps")
    with closing(sb.Spark(shape, w.schedule, weights, max_batch=len(offsets), max_seq_len=96, kv_page_tokens=16)) as sp:
        sp.tune("one_row", 2)
        compare_run(sp, shape, w.schedule, weights, [wl.make_prompt(shape, 20 + 9 * b, seed=68 + b) for b in range(len(offsets))], list(offsets),
                    steps, check_kv_every=1, label=f"one row above the exit layer {offsets}")


def test_static_scratch(sb):
    """the words lie in the library's own scratch area too, which holds what another context has left"""
    shape = _shape("static", d_model=776, n_q_heads=7, n_kv_heads=1, d_ffn=1400)
    weights = wl.make_weights(shape, seed=4, gain_std=0.1)
    say("one row on the static scratch area")
    out = []
    for static in (True, False, True):
        with closing(sb.Spark(shape, wl.TINY.schedule, weights, max_batch=1, max_seq_len=96, kv_page_tokens=16, static_scratch=static)) as sp:
            sp.tune("one_row", 2)
            sid = sp.seq_open(0)
            sp.prefill(sid, wl.make_prompt(shape, 2, seed=69))
            out.append((*sp.decode(14, [sid]), sp.get_logits(sid)[0], *sp.get_kv(sid, 3, 12)))
            assert _last_error(sp) == ""
    for o in out[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(o, out[0], strict=True))


def test_two_contexts_on_two_threads(sb):
    """launches of which each has the whole chip, on two streams at once: each thread's results are those it gets alone"""
    import threading

    import torch
    shape = _shape("threads", d_model=1024, n_q_heads=16, n_kv_heads=8, d_ffn=1536)
    weights = wl.make_weights(shape, seed=4, gain_std=0.1)
    say("one row on two threads")

    def go(stream):
        with closing(sb.Spark(shape, wl.TINY.schedule, weights, max_batch=1, max_seq_len=192, kv_page_tokens=64, stream=stream)) as sp:
            sp.tune("one_row", 2)
            sid = sp.seq_open(0)
            sp.prefill(sid, wl.make_prompt(shape, 50, seed=62))
            return np.concatenate([sp.decode(10, [sid])[0] for _ in range(4)]), sp.get_logits(sid)[0]

    alone, out = go(None), [None, None]

    def thread(i):
        out[i] = go(torch.cuda.Stream())

    threads = [threading.Thread(target=thread, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    for o in out:
        assert o is not None and all(np.array_equal(x, y) for x, y in zip(o, alone))


# the call that meets a wait which runs out begins without and with pending rows; one sequence, and three of which single
# ones run full depth now and then; calls of one step that leave the pending rows alone, or complete them
@pytest.mark.parametrize("first,n_seq,steps", [(0, 1, 9), (4, 1, 9), (5, 1, 9), (4, 3, 9), *((k, 1, 1) for k in range(1, 7))])
def test_waits_that_run_out(sb, first, n_seq, steps):
    """the call runs again as launches per operation, from its start: bit by bit what a context gives that has been told
    to take those for this call, and so does what follows, also for a sequence that had no part in the call"""
    shape = _shape("patience", d_model=1024, n_q_heads=16, n_kv_heads=8, d_ffn=1536)
    weights = wl.make_weights(shape, seed=4, gain_std=0.1)

    def go(patient):
        with closing(sb.Spark(shape, wl.TINY.schedule, weights, max_batch=n_seq + 1, max_seq_len=192, kv_page_tokens=16)) as sp:
            sp.tune("one_row", 2)
            ids = [sp.seq_open(b) for b in range(n_seq + 1)]
            for b, s in enumerate(ids):
                sp.prefill(s, wl.make_prompt(shape, 30 + b, seed=63 + b))
            ids, other = ids[:n_seq], ids[n_seq:]
            out = []
            if first:
                out += list(sp.decode(first, ids))
            assert _last_error(sp) == ""
            if patient:
                sp.tune("one_row", 0)
            else:
                sp.tune("wait_polls", 1)
            out += list(sp.decode(steps, ids))
            assert ("gave up" in _last_error(sp)) == (not patient)
            out += list(sp.decode(8, ids))      # launches per operation in both
            out += list(sp.decode(7, other))
            sp.tune("wait_polls", 0)
            sp.tune("one_row", 2)
            out += list(sp.decode(11, ids + other))
            out += [sp.get_logits(s)[0] for s in ids + other]
            for s in ids + other:
                st = sp.seq_state(s)
                out += [np.array(sorted(st.values()))] + [x for l in range(shape.n_layers) for p in range(28, st["upper_valid"], 3) for x in sp.get_kv(s, l, p)]
        return out

    say(f"one row, waits that run out in {steps} after {first} steps of {n_seq}")
    for x, y in zip(go(False), go(True), strict=True):
        assert np.array_equal(x, y)


# a prompt of two tokens is a pass of one row; prompts of 34 and 514 (32 and 512 rows a pass, the latter in the buffers of
# large passes) end with one, whose context is the passes before it and whose words lie where those left their partial sums
@pytest.mark.parametrize("n,rows", [(2, 0), (34, 32), (514, 512)])
@pytest.mark.parametrize("polls", [0, 1])
def test_prompt_passes_of_one_row(sb, n, rows, polls):
    """against the oracle, cache entries too, also where a wait runs out and the pass runs again"""
    w = wl.TINY
    shape = _shape("one row of a prompt", d_model=776, n_q_heads=7, n_kv_heads=1, d_ffn=1400)
    weights = wl.make_weights(shape, seed=4, gain_std=0.1)
    say(f"one row of a prompt of {n}, {polls} polls")
    with closing(sb.Spark(shape, w.schedule, weights, max_batch=1, max_seq_len=544, kv_page_tokens=16)) as sp:
        sp.tune("one_row", 2)
        sp.tune("wait_polls", polls)
        sp.tune("prefill_rows", rows)
        sid = sp.seq_open(0)
        sp.prefill(sid, wl.make_prompt(shape, n, seed=65))
        assert ("gave up" in _last_error(sp)) == (polls > 0)
        sp.seq_close(sid)
        sp.tune("one_row", 2)
        compare_run(sp, shape, w.schedule, weights, [wl.make_prompt(shape, n, seed=66)], [0], 8, check_kv_every=1, kv_all_positions=n < 100,
                    label=f"one row of a prompt of {n}")

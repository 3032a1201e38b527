"""GPU parity: the HIP path against the CPU oracle, bit for bit, through the C boundary."""
import numpy as np
import pytest

from workloads import grammars, configs
from workloads.rng import stream
from tests.helpers import OracleRun, popcount, load_trajectory
from workloads import vocab as wvocab

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch


def _run_parity(torch, zf, Oracle, grammar, tokens, batch, steps, seed, check_every=1, **engine_kw):
    engine_kw.setdefault("state_cache_entries", -1)      # every step through the kernels unless a test asks for the state cache
    eng = zf.Engine(grammar, tokens, device=0, **engine_kw)
    orc = Oracle(grammar)
    run = OracleRun(orc, tokens, [stream(seed, f"sample[{b}]") for b in range(batch)])
    states = [eng.new_state() for _ in range(batch)]
    d_mask = torch.empty((batch, eng.W), dtype=torch.int32, device="cuda")
    overflow = 0
    for step in range(steps):
        want = run.masks()
        if step % check_every == 0:
            d_mask.fill_(0x5A5A5A5A)
            zf.compute_mask(eng, states, d_mask)
            got = d_mask.cpu().numpy().view(np.uint32)
            overflow += eng.mask_report().overflow_chunks
            assert got.shape == want.shape
            if not (got == want).all():
                bad = np.argwhere(got != want)[0]
                w = int(bad[1])
                diff = int(got[bad[0], w]) ^ int(want[bad[0], w])
                v = w * 32 + (diff & -diff).bit_length() - 1
                raise AssertionError(f"step {step} row {bad[0]} token {v} {tokens[v]!r}: gpu={got[bad[0], w]:#x} oracle={want[bad[0], w]:#x}")
        toks = run.step(want)
        for b, t in enumerate(toks):
            if t < 0:
                states[b].reset()
            else:
                states[b].advance(t)
            assert states[b].accepting() == run.states[b].accepting()
    return overflow


MODES = {"automaton": 0, "trie-walk": 1, "store": 2}     # zf_options.walk_mode: all three mask kernels must give the oracle's bits


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("cache", [True, False], ids=["token-mask-cache", "parser-only"])
def test_config1_json_v2k_all_steps(cache, mode, torch_cuda, oracle_lib):
    import paper_2506_01151_amd as zf
    cfg = configs.CONFIGS[1]
    _run_parity(torch_cuda, zf, oracle_lib.Oracle, cfg.grammar(), cfg.vocab(), cfg.batch, cfg.steps, cfg.seed, token_mask_cache=cache, walk_mode=MODES[mode])


@pytest.mark.parametrize("mode", list(MODES))
def test_config2_json_v32k(mode, torch_cuda, oracle_lib):
    import paper_2506_01151_amd as zf
    cfg = configs.CONFIGS[2]
    _run_parity(torch_cuda, zf, oracle_lib.Oracle, cfg.grammar(), cfg.vocab(), cfg.batch, cfg.steps, cfg.seed, walk_mode=MODES[mode])


# the item budget bounds one set under construction (automaton) or the sets of one trie path (trie walk)
@pytest.mark.parametrize("mode,cap", [("automaton", 1), ("automaton", 2), ("automaton", 3), ("trie-walk", 1), ("trie-walk", 2), ("trie-walk", 4), ("trie-walk", 7)])
def test_forced_overflow_gives_same_bits(mode, cap, torch_cuda, oracle_lib):
    """A tiny LDS item budget pushes work to the global-memory fallback; the bits must not change."""
    import paper_2506_01151_amd as zf
    cfg = configs.CONFIGS[1]
    ov = _run_parity(torch_cuda, zf, oracle_lib.Oracle, cfg.grammar(), cfg.vocab(), 2, 24, cfg.seed + 77, lane_item_cap=cap, walk_mode=MODES[mode])
    assert ov > 0, "the cap was meant to force the fallback pass"


@pytest.mark.parametrize("seed", range(16))
def test_random_grammars(seed, torch_cuda, oracle_lib):
    """Seeded random grammars (empty rules, unit cycles, all kinds of recursion, ambiguity): both mask
    kernels against the oracle at every step, once with the default item budget and once with a
    budget of two or three items that sends much of the work through the fallback pass."""
    import paper_2506_01151_amd as zf
    from workloads import random_grammars
    g = random_grammars.random_grammar(seed)
    toks = random_grammars.random_vocab(seed, 400)
    for mode in MODES.values():
        _run_parity(torch_cuda, zf, oracle_lib.Oracle, g, toks, 3, 20, 1000 + seed, walk_mode=mode)
        if mode != 2:     # a budget of two or three items: the per-block kernels hand such sets to the fallback pass
            _run_parity(torch_cuda, zf, oracle_lib.Oracle, g, toks, 2, 12, 2000 + seed, lane_item_cap=3 - mode, token_mask_cache=seed % 2 == 0, walk_mode=mode)
        else:
            _run_parity(torch_cuda, zf, oracle_lib.Oracle, g, toks, 2, 12, 2000 + seed, token_mask_cache=seed % 2 == 0, walk_mode=mode)


def test_overflow_beyond_the_fallback_is_an_error(torch_cuda):
    """When even the fallback arena is too small the call must fail loudly (no silent wrong mask)."""
    import paper_2506_01151_amd as zf
    cfg = configs.CONFIGS[1]
    eng = zf.Engine(cfg.grammar(), cfg.vocab(), device=0, lane_item_cap=1, fallback_item_cap=1)
    s = eng.new_state()
    s.advance_bytes(b'{"a": [1')
    d_mask = torch_cuda.empty((1, eng.W), dtype=torch_cuda.int32, device="cuda")
    with pytest.raises(zf.ZfError) as ei:
        zf.compute_mask(eng, [s], d_mask)
    assert ei.value.code == zf.ZF_ERR_OVERFLOW


@pytest.mark.parametrize("chunk", [8, 16, 32])
def test_chunk_sizes(chunk, torch_cuda, oracle_lib):
    import paper_2506_01151_amd as zf
    cfg = configs.CONFIGS[1]
    _run_parity(torch_cuda, zf, oracle_lib.Oracle, cfg.grammar(), cfg.vocab(2048 - 37), 3, 32, cfg.seed + 5, chunk_strings=chunk)


def _replay_all_rows(torch, zf, oracle_lib, idx, variants, stride_of=None):
    """Replay configuration idx's oracle-sampled trajectory at its full batch and vocabulary on the oracle and on one
    engine per variant; at every step every row of every variant's mask is compared with the oracle's (variants named
    in stride_of only at every stride-th step and at the last one)."""
    cfg = configs.CONFIGS[idx]
    toks = cfg.vocab()
    off, data = wvocab.vocab_csr(toks)
    rows, steps = cfg.batch, cfg.steps
    traj = load_trajectory(idx, rows, steps)
    g = cfg.grammar()
    orc = oracle_lib.Oracle(g)
    so = [orc.new_state() for _ in range(rows)]
    engines = {name: zf.Engine(g, toks, device=0, state_cache_entries=-1, **kw) for name, kw in variants.items()}
    batches = {name: zf.StateBatch([e.new_state() for _ in range(rows)]) for name, e in engines.items()}
    d_mask = torch.empty((rows, engines[next(iter(engines))].W), dtype=torch.int32, device="cuda")
    n_checked = {name: 0 for name in engines}
    for step, ids in enumerate(traj):
        for b, t in enumerate(ids):
            if t < 0:
                so[b] = orc.new_state()
            else:
                assert so[b].feed_bytes(toks[t])
        want = np.stack([s.mask(off, data, 16) for s in so])
        for name, eng in engines.items():
            batches[name].advance(ids)
            if stride_of and name in stride_of and step % stride_of[name] and step != steps - 1:
                continue
            d_mask.fill_(-1)
            zf.compute_mask(eng, batches[name], d_mask)
            got = d_mask.cpu().numpy().view(np.uint32)
            if not np.array_equal(got, want):
                b = int(np.argwhere((got != want).any(axis=1))[0][0])
                raise AssertionError(f"cfg{idx} {name} step {step} row {b}")
            n_checked[name] += rows
    return n_checked, rows * steps


def test_config3_every_step_every_row(torch_cuda, oracle_lib):
    """Configuration 3 at its stated shape (16 rows x 512 steps, V = 128,256): all three mask kernels against the oracle at
    every step on every row; with the token-mask cache off (every token through the parser) at every 4th step."""
    import paper_2506_01151_amd as zf
    variants = {"store": dict(walk_mode=2), "automaton": dict(walk_mode=0), "trie-walk": dict(walk_mode=1), "store-parser-only": dict(walk_mode=2, token_mask_cache=False),
                "automaton-parser-only": dict(walk_mode=0, token_mask_cache=False), "trie-walk-parser-only": dict(walk_mode=1, token_mask_cache=False)}
    n, full = _replay_all_rows(torch_cuda, zf, oracle_lib, 3, variants, {"automaton-parser-only": 4, "trie-walk-parser-only": 4, "store-parser-only": 4})
    assert n["store"] == full == 16 * 512 and n["automaton"] == full and n["trie-walk"] == full


def test_config4_every_step_every_row(torch_cuda, oracle_lib):
    """Configuration 4 at its stated shape (64 rows x 256 steps, V = 128,256): all three mask kernels, every step, every row."""
    import paper_2506_01151_amd as zf
    n, full = _replay_all_rows(torch_cuda, zf, oracle_lib, 4, {"store": dict(walk_mode=2), "automaton": dict(walk_mode=0), "trie-walk": dict(walk_mode=1)})
    assert n["store"] == full == 64 * 256 and n["automaton"] == full and n["trie-walk"] == full


CFG5_CHECK_STEPS = 12      # steps of the trajectory at which masks are compared (spread evenly, the last one included) ...
CFG5_CHECK_ROWS = 6        # ... on this many seeded rows each: the oracle keeps every Earley set, a mask at step 600 costs it about a second


@pytest.mark.parametrize("pruning,mode,token_cache", [(p, m, c) for c in (True, False) for p in (True, False) for m in MODES],
                         ids=[f"{p}-{m}{c}" for c in ("", "-parser-only") for p in ("pruned", "unpruned") for m in MODES])
def test_config5_full_batch_pruning_on_and_off(pruning, mode, token_cache, torch_cuda, oracle_lib):
    """Configuration 5 at its stated batch and vocabulary (64 rows, V = 152,064) along the oracle-sampled trajectory, as far
    as the file goes: one compute_mask call covers all 64 rows (the launch shape the benchmark times); a seeded, reported
    subsample of (step, row) pairs is compared bit for bit with the oracle, with ZapFormat pruning on and off, every mask kernel (with pruning off the persistent automaton is not used: calls that
    the token-mask cache decides, as it does every one of this configuration, go through the look-ups' kernel, others through the per-block automaton), with every token left to the parser as well."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[5]
    toks = cfg.vocab()
    off, data = wvocab.vocab_csr(toks)
    rows = cfg.batch
    traj = load_trajectory(5, rows, None)
    steps = len(traj)
    assert steps >= 256
    g = cfg.grammar()
    eng = zf.Engine(g, toks, device=0, pruning=pruning, state_cache_entries=-1, walk_mode=MODES[mode], token_mask_cache=token_cache)
    orc = oracle_lib.Oracle(g)
    so = [orc.new_state() for _ in range(rows)]
    ss = zf.StateBatch([eng.new_state() for _ in range(rows)])
    d_mask = torch.empty((rows, eng.W), dtype=torch.int32, device="cuda")
    check_at = sorted({(k + 1) * steps // CFG5_CHECK_STEPS - 1 for k in range(CFG5_CHECK_STEPS)} | {0, 7})
    pick = stream(cfg.seed, "parity-rows")
    pairs = []
    for step, ids in enumerate(traj):
        for b, t in enumerate(ids):
            if t < 0:
                so[b] = orc.new_state()
            else:
                assert so[b].feed_bytes(toks[t])
        ss.advance(ids)
        if step in check_at:
            d_mask.fill_(-1)
            zf.compute_mask(eng, ss, d_mask)
            got = d_mask.cpu().numpy().view(np.uint32)
            for b in sorted({pick.below(rows) for _ in range(CFG5_CHECK_ROWS)}):
                assert (got[b] == so[b].mask(off, data, 16)).all(), f"cfg5 step {step} row {b}"
                assert ss[b].accepting() == so[b].accepting()
                pairs.append((step, b))
    print(f"config 5 {'pruned' if pruning else 'unpruned'} {mode}: {steps} steps x {rows} rows replayed, compared (step, row): {pairs}")
    assert len(pairs) >= 40


LONG5 = [  # pruning, mask kernel, sentences with one long sum at the top level, compare every
    (True, "store", True, 8),
    (True, "store", False, 8),
    (True, "automaton", False, 16),
    (True, "trie-walk", False, 32),
    (False, "automaton", False, 32),
]


@pytest.mark.parametrize("pruning,mode,flat,every", LONG5, ids=[f"{'pruned' if p else 'unpruned'}-{m}-{'long-sums' if f else 'nested-groups'}" for p, m, f, _ in LONG5])
def test_config5_all_1024_steps_against_the_language_description(pruning, mode, flat, every, torch_cuda, oracle_lib):
    """Configuration 5 at its stated shape to its last decode step: 64 rows x 1,024 steps, V = 152,064.  The oracle-sampled
    trajectory ends at step 296 (the oracle keeps every Earley set of an ambiguous grammar: a mask at step 1,000 costs it
    minutes), so the rows here follow seeded sentences of the expression language cut into vocabulary tokens (valid by
    construction, workloads/sentences.py), and the masks of ALL 64 rows are compared, at every `every`-th step and at the last
    one, with the description of the language's viable prefixes in tests/expr_language.py, which the Earley oracle pins on short
    prefixes (tests/test_oracle_pins.py) and, here, on two rows at the full vocabulary during the first steps.  Two shapes of
    sentence: one long sum at the top level (every operator is another way to split it: even the pruned chart reaches 20,000
    items, which only the persistent automaton's kernel is asked to take), and nested groups of two to four operands (pruned
    charts of tens of items against 9,000 unpruned: every mask kernel, pruning on and off)."""
    import paper_2506_01151_amd as zf
    from tests.expr_language import ExprLanguage, ExprRow
    from workloads.sentences import expr_sentence, cut_into_tokens
    torch = torch_cuda
    cfg = configs.CONFIGS[5]
    toks = cfg.vocab()
    off, data = wvocab.vocab_csr(toks)
    rows, steps = cfg.batch, cfg.steps
    seqs = [cut_into_tokens(toks, expr_sentence(cfg.seed, f"sentence[{b}]", 4 * steps + 64, flat=flat), steps) for b in range(rows)]
    assert all(len(q) == steps for q in seqs)
    lang = ExprLanguage(toks)
    want_rows = [ExprRow() for _ in range(rows)]
    eng = zf.Engine(cfg.grammar(), toks, device=0, pruning=pruning, state_cache_entries=-1, walk_mode=MODES[mode])
    ss = zf.StateBatch([eng.new_state() for _ in range(rows)])
    orc = oracle_lib.Oracle(cfg.grammar())
    so = {b: orc.new_state() for b in (3, 40)}
    d_mask = torch.empty((rows, eng.W), dtype=torch.int32, device="cuda")
    n_checked = 0
    for step in range(steps):
        ids = [seqs[b][step] for b in range(rows)]
        for b in range(rows):
            assert want_rows[b].feed(toks[ids[b]]), (step, b)
        ss.advance(ids)
        if step < 24:
            for b, s in so.items():
                assert s.feed_bytes(toks[ids[b]])
        if step % every == every - 1 or step == steps - 1 or step in (0, 5, 23):
            d_mask.fill_(-1)
            zf.compute_mask(eng, ss, d_mask)
            got = d_mask.cpu().numpy().view(np.uint32)
            for b in range(rows):
                assert (got[b] == lang.mask(want_rows[b].mode, want_rows[b].depth)).all(), f"cfg5 step {step} row {b}"
                assert ss[b].accepting() == want_rows[b].accepting(), f"cfg5 step {step} row {b} accepting"
            if step in (0, 5, 23):
                for b, s in so.items():
                    assert (got[b] == s.mask(off, data, 16)).all(), f"cfg5 oracle step {step} row {b}"
            n_checked += rows
    print(f"config 5 {'pruned' if pruning else 'unpruned'} {mode}: {steps} steps x {rows} rows, {n_checked} masks compared")
    assert n_checked >= rows * (steps // every)


STATE_CACHE = [  # config, rows, steps, compare every, cache rows (0 = default), expect the cache to be used
    (3, 16, 512, 29, 0, True),
    (3, 16, 512, 41, 32, True),     # the smallest cache a batch of 16 may use: constant eviction
    (3, 16, 128, 17, 16, False),    # too small for the batch: bypassed
    (4, 64, 256, 37, 256, True),
]


@pytest.mark.parametrize("idx,rows,steps,every,entries,used", STATE_CACHE, ids=[f"cfg{r[0]}-{r[4] or 'default'}" for r in STATE_CACHE])
def test_state_cache_replay(idx, rows, steps, every, entries, used, torch_cuda, oracle_lib):
    """State cache (Section 5.2) on: compute_mask at every step of the trajectory, so that rows are
    served from cached masks as in real decoding; at sampled steps every row equals the oracle."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[idx]
    toks = cfg.vocab()
    off, data = wvocab.vocab_csr(toks)
    traj = load_trajectory(idx, rows, steps)
    g = cfg.grammar()
    eng = zf.Engine(g, toks, device=0, state_cache_entries=entries)
    orc = oracle_lib.Oracle(g)
    so = [orc.new_state() for _ in range(rows)]
    ss = [eng.new_state() for _ in range(rows)]
    d_mask = torch.empty((rows, eng.W), dtype=torch.int32, device="cuda")
    hits = misses = 0
    for step, ids in enumerate(traj):
        for b, t in enumerate(ids):
            if t < 0:
                so[b] = orc.new_state()
                ss[b].reset()
            else:
                assert so[b].feed_bytes(toks[t])
                ss[b].advance(t)
        d_mask.fill_(0x33333333)
        zf.compute_mask(eng, ss, d_mask)
        r = eng.mask_report()
        assert r.cache_hits + r.cache_misses == (rows if used else 0)
        hits += r.cache_hits
        misses += r.cache_misses
        if step % every == 0 or step == steps - 1:
            got = d_mask.cpu().numpy().view(np.uint32)
            for b in range(rows):
                want = so[b].mask(off, data, 16)
                assert (got[b] == want).all(), f"cfg{idx} step {step} row {b} (hits so far {hits}, misses {misses})"
    if used:
        assert hits > misses > 0


def test_state_cache_rows_in_one_call_and_clearing(torch_cuda, oracle_lib):
    """Equal rows of one call are computed once; clearing the cache makes the next call start cold;
    a failed call leaves nothing behind that a later call could be served from."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[2]
    toks = cfg.vocab()
    off, data = wvocab.vocab_csr(toks)
    g = cfg.grammar()
    eng = zf.Engine(g, toks, device=0)
    orc = oracle_lib.Oracle(g)
    o = orc.new_state()
    assert o.feed_bytes(b'{"key": [1, {"x": "a')
    want = o.mask(off, data, 4)
    ss = [eng.new_state() for _ in range(8)]
    for s in ss:
        s.advance_bytes(b'{"key": [1, {"x": "a')
    d_mask = torch.empty((8, eng.W), dtype=torch.int32, device="cuda")
    for expect in [(7, 1), (8, 0), None, (7, 1)]:
        if expect is None:
            eng.clear_state_cache()
            continue
        d_mask.fill_(0)
        zf.compute_mask(eng, ss, d_mask)
        r = eng.mask_report()
        assert (r.cache_hits, r.cache_misses) == expect
        assert (d_mask.cpu().numpy().view(np.uint32) == want[None, :]).all()
    # same prefix through an engine whose budgets are too small: the error must not poison its cache
    tiny = zf.Engine(g, toks, device=0, lane_item_cap=1, fallback_item_cap=1)
    t = tiny.new_state()
    t.advance_bytes(b'{"a": [1')
    for _ in range(2):
        with pytest.raises(zf.ZfError) as ei:
            zf.compute_mask(tiny, [t], d_mask[:1])
        assert ei.value.code == zf.ZF_ERR_OVERFLOW
        assert tiny.mask_report().cache_misses == 1


def test_async_calls_match_the_waiting_call(torch_cuda, oracle_lib):
    """compute_mask_async + mask_wait: several calls in flight on one stream, apply_mask queued right
    behind each; results equal the waiting call's and the oracle's; a fifth call in flight is refused;
    an overflow beyond the fallback arena surfaces in mask_wait."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    cfg = configs.CONFIGS[2]
    toks = cfg.vocab()
    off, data = wvocab.vocab_csr(toks)
    g = cfg.grammar()
    eng = zf.Engine(g, toks, device=0)
    orc = oracle_lib.Oracle(g)
    prefixes = [b'{"a', b'[1, 2', b' {"k": "\\', b"tr"]
    so, ss = [], []
    for p in prefixes:
        a, b = orc.new_state(), eng.new_state()
        assert a.feed_bytes(p)
        b.advance_bytes(p)
        so.append(a)
        ss.append(b)
    masks = [torch.full((1, eng.W), -1, dtype=torch.int32, device="cuda") for _ in prefixes]
    logits = configs.make_logits(cfg, 3, device="cuda", batch=1)
    outs = [torch.empty_like(logits) for _ in prefixes]
    for i in range(4):
        zf.compute_mask_async(eng, [ss[i]], masks[i])
        zf.apply_mask(eng, logits, masks[i], out=outs[i])
    with pytest.raises(zf.ZfError) as ei:
        zf.compute_mask_async(eng, [ss[0]], masks[0])
    assert ei.value.code == zf.ZF_ERR_INVALID_ARG
    zf.mask_wait(eng)
    lbits = logits.view(torch.int32).cpu().numpy().view(np.uint32)
    for i in range(4):
        want = so[i].mask(off, data, 4)
        assert (masks[i].cpu().numpy().view(np.uint32)[0] == want).all(), prefixes[i]
        assert outs[i].view(torch.int32).cpu().numpy().view(np.uint32).tobytes() == oracle_apply(lbits, want[None, :]).tobytes()
    tiny = zf.Engine(g, toks, device=0, lane_item_cap=1, fallback_item_cap=1)
    s = tiny.new_state()
    s.advance_bytes(b'{"a": [1')
    zf.compute_mask_async(tiny, [s], masks[0])
    with pytest.raises(zf.ZfError) as ei:
        zf.mask_wait(tiny)
    assert ei.value.code == zf.ZF_ERR_OVERFLOW


def test_persistent_automaton_bookkeeping(torch_cuda, oracle_lib):
    """The persistent automaton (walk_mode 2) keeps, per state, where the row stands in the device's store and which
    bytes were fed since.  Calls in flight while rows move on, a cleared store (rows come back in through their charts),
    a row fed more bytes than a call carries, clones, resets and a state destroyed while a call is in flight: the masks
    equal the oracle's every time, and a repeated call takes no Earley step at all."""
    import gc
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[2]
    toks = cfg.vocab()
    off, data = wvocab.vocab_csr(toks)
    g = cfg.grammar()
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=2)
    orc = oracle_lib.Oracle(g)
    rows = 6
    run = OracleRun(orc, toks, [stream(99, f"book[{b}]") for b in range(rows)])
    ss = zf.StateBatch([eng.new_state() for _ in range(rows)])

    def check(states, oracle_states, what):
        d = torch.full((len(states), eng.W), -1, dtype=torch.int32, device="cuda")
        zf.compute_mask(eng, states, d)
        got = d.cpu().numpy().view(np.uint32)
        for b, o in enumerate(oracle_states):
            assert (got[b] == o.mask(off, data, 8)).all(), (what, b)

    for _ in range(10):                                    # get going
        ss.advance(run.step(run.masks()))
    check(ss, run.states, "start")
    # four calls in flight, the rows advancing in between: each call walks what was fed since the last state the host knew of
    masks = [torch.full((rows, eng.W), -1, dtype=torch.int32, device="cuda") for _ in range(4)]
    want = []
    for k in range(4):
        ss.advance(run.step(run.masks()))
        want.append(run.masks())
        zf.compute_mask_async(eng, ss, masks[k])
    zf.mask_wait(eng)
    torch.cuda.synchronize()
    for k in range(4):
        assert (masks[k].cpu().numpy().view(np.uint32) == want[k]).all(), f"call {k} in flight"
    # the same states again: everything is in the table
    check(ss, run.states, "repeat")
    assert eng.mask_report().parser_steps == 0
    # the store cleared: the rows come back in from their host charts
    eng.clear_state_cache()
    check(ss, run.states, "after clearing the store")
    for _ in range(3):
        ss.advance(run.step(run.masks()))
    check(ss, run.states, "three steps after clearing")
    # a row fed far more bytes than a call carries
    long_o, long_s = orc.new_state(), eng.new_state()
    text = b'{"k": "' + b"abc def " * 700
    assert long_o.feed_bytes(text)
    long_s.advance_bytes(text)
    check([long_s], [long_o], "5,600 bytes at once")
    long_s.advance_bytes(b'", "n": [1, 2')
    assert long_o.feed_bytes(b'", "n": [1, 2')
    check([long_s], [long_o], "and a few more")
    # clones go their own ways; a reset row starts over
    c_s, c_o = ss[0].clone(), run.states[0].clone()
    m = c_o.mask(off, data, 8)
    t = next(v for v in range(300, len(toks)) if (m[v >> 5] >> (v & 31)) & 1)
    c_s.advance(t)
    assert c_o.feed_bytes(toks[t])
    check([c_s, ss[0]], [c_o, run.states[0]], "clone")
    ss[1].reset()
    run.states[1] = orc.new_state()
    check(ss, run.states, "reset")
    # a state destroyed while a call that names it is in flight
    doomed = eng.new_state()
    doomed.advance_bytes(b"[1, ")
    d2 = torch.full((2, eng.W), -1, dtype=torch.int32, device="cuda")
    zf.compute_mask_async(eng, [doomed, ss[0]], d2)
    del doomed
    gc.collect()
    zf.mask_wait(eng)
    torch.cuda.synchronize()
    assert (d2.cpu().numpy().view(np.uint32)[1] == run.states[0].mask(off, data, 8)).all()
    check(ss, run.states, "afterwards")


@pytest.mark.parametrize("cap", [2, 40], ids=["budget-2", "budget-40"])
def test_persistent_automaton_out_of_room(cap, torch_cuda, oracle_lib):
    """A set that outgrows a wavefront's scratch fails the call on the persistent automaton; the waiting call then answers
    through the per-block automaton and its fallback pass, the following calls go that way too for a while, and the masks
    are the oracle's throughout.  The call that does not wait reports the overflow from mask_wait."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[5]
    g, toks = cfg.grammar(), cfg.vocab(6000)
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=2, lane_item_cap=cap)
    prefixes = [b"a" + b"+b" * 30, b"(x*y" + b"+(z)" * 12, b"q"]
    so, ss = [], []
    for p in prefixes:
        a, b = orc.new_state(), eng.new_state()
        assert a.feed_bytes(p)
        b.advance_bytes(p)
        so.append(a)
        ss.append(b)
    d_mask = torch.full((len(ss), eng.W), -1, dtype=torch.int32, device="cuda")
    for rep in range(12):                                  # beyond the first back-off of 8 calls: the store is tried again, fails again
        d_mask.fill_(-1)
        zf.compute_mask(eng, ss, d_mask)
        got = d_mask.cpu().numpy().view(np.uint32)
        for i, a in enumerate(so):
            assert (got[i] == a.mask(off, data, 4)).all(), (rep, prefixes[i][:8])
    fresh = zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=2, lane_item_cap=cap)
    s = fresh.new_state()
    s.advance_bytes(prefixes[0])
    zf.compute_mask_async(fresh, [s], d_mask[:1])
    with pytest.raises(zf.ZfError) as ei:
        zf.mask_wait(fresh)
    assert ei.value.code == zf.ZF_ERR_OVERFLOW
    zf.compute_mask(fresh, [s], d_mask[:1])                # and the engine goes on working
    assert (d_mask[:1].cpu().numpy().view(np.uint32)[0] == so[0].mask(off, data, 4)).all()


def test_edge_cases(torch_cuda, oracle_lib):
    """Empty tokens, duplicates, a vocabulary smaller than one word, rows in different states,
    a finished sentence (empty mask), V not a multiple of 32."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g = grammars.json_grammar()
    orc = oracle_lib.Oracle(g)
    for toks in ([b"", b"1", b"1", b"", b"[", b"]", b"[]", b" ", b"x"],
                 [b'"', b""] * 20 + [bytes([c]) for c in range(256)] + [b"tru", b"true", b"e", b'{"a":1}', b"}"]):
        off, data = wvocab.vocab_csr(toks)
        eng = zf.Engine(g, toks, device=0)
        prefixes = [b"", b"[", b"[1", b"[]", b'{"a":1}', b"tr", b'{"k":"\\u12']
        so, ss = [], []
        for p in prefixes:
            a, b = orc.new_state(), eng.new_state()
            assert a.feed_bytes(p)
            b.advance_bytes(p)
            so.append(a)
            ss.append(b)
        d_mask = torch.full((len(prefixes), eng.W), -1, dtype=torch.int32, device="cuda")
        zf.compute_mask(eng, ss, d_mask)
        got = d_mask.cpu().numpy().view(np.uint32)
        for i, a in enumerate(so):
            assert (got[i] == a.mask(off, data, 1)).all(), (toks[:4], prefixes[i])
    # a grammar whose sentence cannot be extended: after the last byte the mask is all zero
    g2 = grammars.w2_grammar()
    toks = [b"a", b"b", b"ab"]
    eng = zf.Engine(g2, toks, device=0)
    s = eng.new_state()
    s.advance(2)
    d_mask = torch.full((1, eng.W), -1, dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, [s], d_mask)
    assert d_mask.cpu().numpy().view(np.uint32).tolist() == [[0]] and s.accepting()


@pytest.mark.parametrize("mode", list(MODES))
def test_long_tokens_deep_nesting_many_classes(mode, torch_cuda, oracle_lib):
    """Tokens longer than the 16 bytes a lane fetches at once, nesting deeper than the automaton's state budget
    (those strings must come back through the fallback pass), and a grammar with more than 64 byte classes."""
    import paper_2506_01151_amd as zf
    from tests.helpers import edge_vocab_json
    torch = torch_cuda
    g = grammars.json_grammar()
    toks = edge_vocab_json()
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=MODES[mode])
    prefixes = [b"", b"[", b'{"k":"', b"[1,", b'[[{"a":[', b'{"k":"v', b"[1", b'["\\']
    so, ss = [], []
    for p in prefixes:
        a, b = orc.new_state(), eng.new_state()
        assert a.feed_bytes(p)
        b.advance_bytes(p)
        so.append(a)
        ss.append(b)
    d_mask = torch.full((len(prefixes), eng.W), -1, dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, ss, d_mask)
    got = d_mask.cpu().numpy().view(np.uint32)
    for i, a in enumerate(so):
        assert (got[i] == a.mask(off, data, 4)).all(), prefixes[i]
    if mode == "automaton":
        assert eng.mask_report().overflow_chunks > 0, "runs of 120 brackets were meant to outgrow the state budget"
    if mode == "store":
        assert eng.mask_report().overflow_chunks == 0      # the persistent automaton has room for every nesting depth
    g2 = grammars.many_classes_grammar(100)
    toks2 = [bytes([c]) for c in range(256)] + [bytes([32 + c, 32 + (c * 7 + 3) % 100]) for c in range(100)] + [bytes([32 + c, 32 + (c * 7 + 3) % 100, 32 + (c * 5) % 100]) for c in range(100)]
    assert zf.Engine(g2, toks2, device=-1).info.n_byte_classes > 64
    _run_parity(torch, zf, oracle_lib.Oracle, g2, toks2, 3, 12, 4242, walk_mode=MODES[mode])


def test_exploration_at_compile_time_changes_no_mask(torch_cuda, oracle_lib):
    """zf_options.precompute_states: the automaton explored from the empty prefix when the engine is compiled and
    whenever it is emptied.  A grammar without recursion (the W2 sequence, a JSON schema with fixed keys cut short
    by its budget) and a recursive one; masks against the oracle with the exploration on, off, and after the engine
    has been emptied in mid-sentence; and the first steps of a decode loop find more of their transitions
    computed with it than without."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[2]
    g, toks = cfg.grammar(), cfg.vocab()
    for pre in (-1, 64, 0):
        _run_parity(torch, zf, oracle_lib.Oracle, g, toks, 4, 24, 991, walk_mode=2, precompute_states=pre)
    _run_parity(torch, zf, oracle_lib.Oracle, grammars.w2_grammar(), [b"a", b"b", b"ab", b"ba", b""], 2, 6, 5, walk_mode=2)
    cfg3 = configs.CONFIGS[3]
    g3, toks3 = cfg3.grammar(), cfg3.vocab(8000)
    steps_taken = {}
    for pre in (-1, 0):
        eng = zf.Engine(g3, toks3, device=0, state_cache_entries=-1, walk_mode=2, precompute_states=pre)
        orc = oracle_lib.Oracle(g3)
        run = OracleRun(orc, toks3, [stream(77, f"sample[{b}]") for b in range(4)])
        states = [eng.new_state() for _ in range(4)]
        d_mask = torch.empty((4, eng.W), dtype=torch.int32, device="cuda")
        total = 0
        for step in range(12):
            want = run.masks()
            zf.compute_mask(eng, states, d_mask)
            total += eng.mask_report().parser_steps
            assert (d_mask.cpu().numpy().view(np.uint32) == want).all(), (pre, step)
            if step == 6:
                eng.clear_state_cache()                     # emptied (and explored again) under the rows' feet
            for b, t in enumerate(run.step(want)):
                states[b].reset() if t < 0 else states[b].advance(t)
        steps_taken[pre] = total
    assert steps_taken[0] < steps_taken[-1], steps_taken


@pytest.mark.parametrize("pre", [1, 2, 33, 1025, 0], ids=lambda p: f"budget-{p}")
@pytest.mark.parametrize("cfg_id", [2, 5])
def test_store_filled_from_the_host_automaton(cfg_id, pre, torch_cuda, oracle_lib):
    """Where the exploration's budget ends, the device goes on by itself from states the host has filled in: a budget of one state,
    budgets in the middle of a block of states and just beyond one, and the default; recursive grammars, one of them ambiguous
    (sets the host and the device make in different orders have one name)."""
    import paper_2506_01151_amd as zf
    cfg = configs.CONFIGS[cfg_id]
    _run_parity(torch_cuda, zf, oracle_lib.Oracle, cfg.grammar(), cfg.vocab(3000), 5, 14, 4711, walk_mode=2, precompute_states=pre)


@pytest.mark.parametrize("cap", [None, 72, 200], ids=["default-budget", "budget-72", "budget-200"])
def test_wide_sets_of_an_ambiguous_grammar(cap, torch_cuda, oracle_lib):
    """Sets far beyond 64 items (the ambiguous expression grammar after sums of 20 to 150 operands: every
    operand is another origin) through the mask automaton: the set under construction then lives in LDS
    behind a hash table and Complete deals the origin sets' items to the lanes.  With a budget of 72 or
    200 items the wider sets run out of room and their strings must come back through the fallback pass."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[5]
    g, toks = cfg.grammar(), cfg.vocab(6000)
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    kw = {} if cap is None else {"lane_item_cap": cap}
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, **kw)
    prefixes = [b"a" + b"+b" * 20, b"a" + b"*77" * 45 + b"+", b"(a" + b"+b" * 70 + b")*c" + b"+d" * 12, b"x" + b"+(y)" * 150, b"q" + b"*r" * 160 + b"*(",
                b"a+b", b"a" + b"+b" * 300]
    so, ss = [], []
    for p in prefixes:
        a, b = orc.new_state(), eng.new_state()
        assert a.feed_bytes(p)
        b.advance_bytes(p)
        so.append(a)
        ss.append(b)
    def last_set_size(st):
        items, n_sets = st.chart()
        return sum(1 for it in items if it[0] == n_sets - 1)
    assert max(last_set_size(s) for s in ss) > 250
    d_mask = torch.full((len(prefixes), eng.W), -1, dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, ss, d_mask)
    got = d_mask.cpu().numpy().view(np.uint32)
    for i, a in enumerate(so):
        assert (got[i] == a.mask(off, data, 4)).all(), prefixes[i][:12]
    if cap is not None:
        assert eng.mask_report().overflow_chunks > 0, "the budget was meant to be too small for the widest sets"


@pytest.mark.parametrize("mode", list(MODES))
def test_many_rows_and_longest_token(mode, torch_cuda, oracle_lib):
    """A batch larger than the number of compute units (one block per row and less) and tokens of the
    maximum length the library takes (255 bytes), valid and invalid ones."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[1]
    g = cfg.grammar()
    toks = cfg.vocab(600) + [b'"' + b"x" * 253 + b'"', b"[" * 255, b"1" * 255, b'"' + b"y" * 254, b" " * 254 + b"}", b"a" * 255]
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=MODES[mode])
    rows = 300
    rs = stream(cfg.seed, "many-rows")
    pieces = [b"", b"[", b'{"a":', b'{"a": "', b"[1, 2", b'[{"k": [', b"tr", b'"abc', b"[[[", b'{"k":"v"', b"-1.5e", b'["\\u00']
    so, ss = [], []
    for r in range(rows):
        p = pieces[rs.below(len(pieces))]
        a, b = orc.new_state(), eng.new_state()
        assert a.feed_bytes(p)
        b.advance_bytes(p)
        so.append(a)
        ss.append(b)
    d_mask = torch.full((rows, eng.W), -1, dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, ss, d_mask)
    got = d_mask.cpu().numpy().view(np.uint32)
    for r in range(rows):
        assert (got[r] == so[r].mask(off, data, 4)).all(), r


@pytest.mark.parametrize("mode", ["automaton", "store"])
def test_largest_batch_closing_kernel_loops_over_row_groups(mode, torch_cuda, oracle_lib):
    """4,096 rows (the largest batch a call takes) over a vocabulary of 1,000 tokens: the closing kernel's grid is capped at
    what the chip holds at once, so its blocks loop over the 1,024 row groups; with a budget of one item the per-block
    automaton sends strings through the fallback pass, whose wavefronts the other blocks of that grid wait for."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[1]
    g = cfg.grammar()
    toks = cfg.vocab(1000)
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    kw = {"lane_item_cap": 1} if mode == "automaton" else {}
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=MODES[mode], **kw)
    pieces = [b"", b"[", b'{"a":', b'{"a": "', b"[1, 2", b'[{"k": [', b"tr", b'"abc', b"[[[", b'{"k":"v"', b"-1.5e", b'["\\u00', b"[1.0"]
    want, proto = [], []
    for p in pieces:
        a, b = orc.new_state(), eng.new_state()
        assert a.feed_bytes(p)
        b.advance_bytes(p)
        want.append(a.mask(off, data, 4))
        proto.append(b)
    rows = 4096
    rs = stream(cfg.seed, "largest-batch")
    pick = [rs.below(len(pieces)) for _ in range(rows)]
    ss = [proto[k] for k in pick]                          # a state may be named many times in one call
    d_mask = torch.full((rows, eng.W), -1, dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, ss, d_mask)
    got = d_mask.cpu().numpy().view(np.uint32)
    assert (got == np.stack([want[k] for k in pick])).all()
    if mode == "automaton":
        assert eng.mask_report().overflow_chunks > 0


@pytest.mark.parametrize("cap", [None, 1], ids=["default-budget", "budget-1"])
def test_ragged_vocabulary_many_rows_closing_kernel(cap, torch_cuda, oracle_lib):
    """130 rows (a last group of two) over a vocabulary of 40,037 tokens (not a multiple of 32 or 64): the
    closing kernel then serves long runs of tokens per block from LDS copies of the rows, and the last
    block's run ends inside a mask word.  With an item budget of 1 most strings come back through the
    fallback pass, the closing kernel's first phase, whose wavefronts the other blocks wait for."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[2]
    g = cfg.grammar()
    toks = cfg.vocab(40037)
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    kw = {} if cap is None else {"lane_item_cap": cap}
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, **kw)
    rows = 130
    rs = stream(cfg.seed, "ragged-rows")
    pieces = [b"", b"[", b'{"a":', b'{"a": "', b"[1, 2", b'[{"k": [', b"tr", b'"abc', b"[[[", b'{"k":"v"', b"-1.5e", b'["\\u00', b"[1.0", b'{"k": nul']
    so, ss = [], []
    for r in range(rows):
        p = pieces[rs.below(len(pieces))]
        a, b = orc.new_state(), eng.new_state()
        assert a.feed_bytes(p)
        b.advance_bytes(p)
        so.append(a)
        ss.append(b)
    d_mask = torch.full((rows, eng.W), -1, dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, ss, d_mask)
    got = d_mask.cpu().numpy().view(np.uint32)
    for r in range(rows):
        assert (got[r] == so[r].mask(off, data, 8)).all(), r
    assert got[:, -1].max() < (1 << (40037 % 32)), "padding bits of the last word must be zero"
    if cap is not None:
        assert eng.mask_report().overflow_chunks > 0


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("n_words,word_len,lds_mode", [(1500, 5, 1), (1500, 8, 2)])
def test_grammar_tables_beyond_the_lds_budget(n_words, word_len, lds_mode, mode, torch_cuda, oracle_lib):
    """Grammars whose tables do not fit the kernels' LDS budget: only the small tables staged (mode 1) or
    none (mode 2); the kernels then read the rest from global memory."""
    import paper_2506_01151_amd as zf
    g = grammars.big_tables_grammar(n_words, word_len)
    words = [bytes(t.data) for t in g.terminals if len(t.data) == word_len]
    rs = stream(77, "big-tables-vocab")
    toks = [bytes([c]) for c in range(256)]
    for _ in range(400):
        w = words[rs.below(len(words))]
        k = rs.below(4)
        toks.append(w if k == 0 else (w[:1 + rs.below(word_len - 1)] if k == 1 else (w + b" " if k == 2 else w[2:] + b" " + words[rs.below(len(words))][:3])))
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=MODES[mode])
    assert eng.info.table_lds_mode == lds_mode
    del eng
    _run_parity(torch_cuda, zf, oracle_lib.Oracle, g, toks, 3, 6, 31337, walk_mode=MODES[mode])


def test_apply_mask_full_size_bf16(torch_cuda, oracle_lib):
    """Configuration 3's logits shape [16, 128256] bf16, mask from a real state."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    cfg = configs.CONFIGS[3]
    eng = zf.Engine(cfg.grammar(), cfg.vocab(), device=0)
    rng = np.random.default_rng(5)
    mask = rng.integers(0, 2**32, size=(cfg.batch, eng.W), dtype=np.uint32)
    mask[3] = 0
    mask[4] = 0xFFFFFFFF
    logits = configs.make_logits(cfg, 1, device="cuda")
    d_mask = torch.from_numpy(mask.view(np.int32)).cuda()
    out = torch.empty_like(logits)
    zf.apply_mask(eng, logits, d_mask, out=out)
    bits = logits.view(torch.int16).cpu().numpy().view(np.uint16)
    want = oracle_apply(bits, mask)
    assert out.view(torch.int16).cpu().numpy().view(np.uint16).tobytes() == want.tobytes()


FUSED = [("store", "bf16", 0, True), ("store", "f32", 0, False), ("store", "bf16", 13, False), ("store-state-cache", "f32", 0, True),
         ("automaton", "bf16", 0, False), ("trie-walk", "f32", 0, True)]


@pytest.mark.parametrize("variant,dtype,ragged,in_place", FUSED, ids=[f"{v}-{d}-{'ragged' if r else 'even'}-{'in-place' if i else 'out'}" for v, d, r, i in FUSED])
def test_compute_mask_apply_in_one_call(variant, dtype, ragged, in_place, torch_cuda, oracle_lib):
    """zf_compute_mask_apply_async: the mask and the masked logits of every step against the oracle, bit for bit -- through the
    persistent automaton (one kernel does both), with a vocabulary size that is no multiple of a 16-byte piece, with the state
    cache on and through the other mask kernels (two kernels behind the one call)."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    cfg = configs.CONFIGS[1]
    toks = cfg.vocab(2048 - ragged)
    kw = {"store": dict(walk_mode=2, state_cache_entries=-1), "store-state-cache": dict(walk_mode=2, state_cache_entries=64),
          "automaton": dict(walk_mode=0, state_cache_entries=-1), "trie-walk": dict(walk_mode=1, state_cache_entries=-1)}[variant]
    eng = zf.Engine(cfg.grammar(), toks, device=0, **kw)
    B, V = 5, eng.V
    orc = oracle_lib.Oracle(cfg.grammar())
    run = OracleRun(orc, toks, [stream(cfg.seed + 77, f"sample[{b}]") for b in range(B)])
    states = [eng.new_state() for _ in range(B)]
    d_mask = torch.empty((B, eng.W), dtype=torch.int32, device="cuda")
    rng = np.random.default_rng(5)
    ivt = torch.int32 if dtype == "f32" else torch.int16
    for step in range(40):
        want_mask = run.masks()
        if dtype == "f32":
            bits = rng.integers(0, 2**32, size=(B, V), dtype=np.uint32)
            t = torch.from_numpy(bits.view(np.int32)).cuda().view(torch.float32)
        else:
            bits = rng.integers(0, 2**16, size=(B, V), dtype=np.uint16)
            t = torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)
        out = t if in_place else torch.full_like(t, 1.0)
        d_mask.fill_(0x5A5A5A5A)
        zf.compute_mask_apply_async(eng, states, d_mask, t, out=out)
        zf.mask_wait(eng)
        torch.cuda.synchronize()
        got_mask = d_mask.cpu().numpy().view(np.uint32)
        assert np.array_equal(got_mask, want_mask), f"{variant} step {step}: mask"
        want = oracle_apply(bits, want_mask)
        got = out.view(ivt).cpu().numpy().view(bits.dtype)
        assert got.tobytes() == want.tobytes(), f"{variant} step {step}: masked logits"
        for b, tk in enumerate(run.step(want_mask)):
            states[b].reset() if tk < 0 else states[b].advance(tk)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_apply_mask_bit_exact(dtype, torch_cuda, oracle_lib):
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    cfg = configs.CONFIGS[1]
    toks = cfg.vocab(2048 - 13)           # ragged V: not a multiple of 32 nor of the vector width
    eng = zf.Engine(cfg.grammar(), toks, device=0)
    B, V, W = 5, eng.V, eng.W
    rng = np.random.default_rng(11)
    mask = rng.integers(0, 2**32, size=(B, W), dtype=np.uint32)
    if dtype == "f32":
        bits = rng.integers(0, 2**32, size=(B, V), dtype=np.uint32)
        t = torch.from_numpy(bits.view(np.int32)).cuda().view(torch.float32)
    else:
        bits = rng.integers(0, 2**16, size=(B, V), dtype=np.uint16)
        t = torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)
    d_mask = torch.from_numpy(mask.view(np.int32)).cuda()
    want = oracle_apply(bits, mask)
    out = torch.empty_like(t)
    zf.apply_mask(eng, t, d_mask, out=out)
    ivt = torch.int32 if dtype == "f32" else torch.int16
    got = out.view(ivt).cpu().numpy().view(bits.dtype)
    assert got.tobytes() == want.tobytes()
    zf.apply_mask(eng, t, d_mask)         # in place
    assert t.view(ivt).cpu().numpy().view(bits.dtype).tobytes() == want.tobytes()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V,B,shift", [(3, 2, 0), (9, 3, 1), (257, 7, 0), (2033, 65, 1), (40037, 53, 3), (40037, 640, 1)])
def test_apply_mask_rows_at_any_multiple_of_an_element(V, B, shift, dtype, torch_cuda, oracle_lib):
    """Rows packed one behind the other (no row but the first at a multiple of 16 bytes), the tensor itself beginning `shift`
    elements into an allocation, vocabularies smaller than a piece of 16 bytes and just beyond one; the last tensor is of the size from
    which pieces that nothing is allowed of are not read (most mask words of every other row are empty)."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    toks = [b"a"] * V
    eng = zf.Engine(grammars.w1_grammar(), toks, device=0)
    rng = np.random.default_rng(V + B)
    mask = rng.integers(0, 2**32, size=(B, eng.W), dtype=np.uint32)
    mask[::2] &= np.where(rng.random((len(mask[::2]), eng.W)) < 0.1, 0xFFFFFFFF, 0).astype(np.uint32)
    u, i, f = (np.uint32, torch.int32, torch.float32) if dtype == "f32" else (np.uint16, torch.int16, torch.bfloat16)
    bits = rng.integers(0, np.iinfo(u).max, size=(B, V), dtype=u)
    room = torch.zeros(B * V + shift, dtype=i, device="cuda")
    t = room[shift:].view(f).view(B, V)
    t.view(i).copy_(torch.from_numpy(bits.view(np.int32 if dtype == "f32" else np.int16)))
    zf.apply_mask(eng, t, torch.from_numpy(mask.view(np.int32)).cuda())
    assert t.view(i).cpu().numpy().view(u).tobytes() == oracle_apply(bits, mask).tobytes()


LOOKS = [(31, 1, 1, "f32", 0, True), (33, 3, 1, "bf16", 1, True), (2033, 70, 3, "bf16", 3, True), (2048, 130, 130, "f32", 0, True),
         (6001, 300, 2, "f32", 1, True), (9000, 5, 2, "bf16", 0, False), (9001, 68, 68, "bf16", 7, False)]


@pytest.mark.parametrize("V,B,places,dtype,shift,token_cache", LOOKS, ids=[f"{v}x{b}-in-{p}-{d}-at-{s}-{'' if c else 'parser-only'}" for v, b, p, d, s, c in LOOKS])
def test_states_met_before(V, B, places, dtype, shift, token_cache, torch_cuda, oracle_lib):
    """The calls at states whose vocabulary has been walked before (mask_look_kernel), mask and masked logits against the oracle: one
    state with up to 130 rows and more states than travel in the argument block (64), vocabularies below one word and just beyond
    one, rows of logits at any multiple of an element, tokens of up to 123 bytes (15 are at hand), and every token undecided.  The
    rows of a second call stand in the states of the first in another order, so that no row finds its own mask in the tensor."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    from tests.helpers import edge_vocab_json
    torch = torch_cuda
    toks = edge_vocab_json()[::-1] + configs.CONFIGS[2].vocab(max(V, 31))
    toks = toks[:V]
    off, data = wvocab.vocab_csr(toks)
    g = grammars.json_grammar()
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, token_mask_cache=token_cache, precompute_states=-1)
    prefixes = [b"[" * (k // 2) + (b'{"a": ' if k & 1 else b"") for k in range(places)]
    want = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
    rng = np.random.default_rng(V + B)
    u, i, f = (np.uint32, torch.int32, torch.float32) if dtype == "f32" else (np.uint16, torch.int16, torch.bfloat16)
    rows = [eng.new_state() for _ in range(B)]
    for call in range(3):
        at = (np.arange(B) + 7 * call) % places
        for s, p in zip(rows, at):
            s.reset()
            s.advance_bytes(prefixes[p])
        bits = rng.integers(0, np.iinfo(u).max, size=(B, V), dtype=u)
        room = torch.zeros(B * V + shift, dtype=i, device="cuda")
        t = room[shift:].view(f).view(B, V)
        t.view(i).copy_(torch.from_numpy(bits.view(np.int32 if dtype == "f32" else np.int16)))
        d_mask = torch.full((B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        zf.compute_mask_apply_async(eng, rows, d_mask, t)
        zf.mask_wait(eng)
        torch.cuda.synchronize()
        wanted = np.stack([want[p] for p in at])
        assert np.array_equal(d_mask.cpu().numpy().view(np.uint32), wanted), call
        assert t.view(i).cpu().numpy().view(u).tobytes() == oracle_apply(bits, wanted).tobytes(), call


@pytest.mark.parametrize("V,B,places,dtype,shift", [(2033, 16, 1, "bf16", 0), (33, 17, 1, "bf16", 1), (6001, 35, 2, "bf16", 3), (2049, 128, 1, "f32", 1), (2047, 129, 1, "f32", 0),
                                                    (4097, 256, 1, "bf16", 5), (4096, 257, 1, "bf16", 0)])
def test_rows_of_large_groups(V, B, places, dtype, shift, torch_cuda, oracle_lib):
    """Groups around the sizes from which on the wavefronts that mask the logits store the mask rows (17 bf16 rows, 129 fp32), with all rows of the argument block and one more."""
    test_states_met_before(V, B, places, dtype, shift, True, torch_cuda, oracle_lib)


@pytest.mark.parametrize("n", [1, 15, 17, 64, 65, 257, 1024, 1500])
def test_rows_of_large_groups_without_logits(n, torch_cuda):
    """Waiting calls whose rows all stand in one state: the more rows, the fewer words a wavefront takes; every row is the row of a call of its own."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    eng = zf.Engine(grammars.json_grammar(), configs.CONFIGS[2].vocab(6007), device=0, state_cache_entries=-1)
    st = eng.new_state()
    st.advance_bytes(b'{"a": [1')
    want = torch.empty((1, eng.W), dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, [st], want)
    got = torch.full((n + 1, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    for _ in range(2):
        zf.compute_mask(eng, [st] * n, got[:n])
        assert torch.equal(got[:n], want.expand(n, -1)) and bool((got[n] == 0x5A5A5A5A).all())
        got[:n].fill_(0x5A5A5A5A)


@pytest.mark.parametrize("V,B", [(16384, 300), (16385, 300), (33001, 300), (4096, 1), (4097, 3)])
def test_per_block_automaton_passes(V, B, torch_cuda, oracle_lib):
    """The per-block automaton where a row's share of a block is one word less, and more, than a pass takes (512 words; 300 rows have a block
    each), and where a row has hardly a block's worth of words: an ambiguous grammar with pruning off, against the oracle.  Every ninth token ends a group, which
    only the parser knows of, so that strings of every pass are left to it."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[5]
    g, toks = cfg.grammar(), cfg.vocab(V)
    for k in range(0, V, 9):
        n, word = k // 9, b""
        for _ in range(4):
            word, n = word + bytes([97 + n % 26]), n // 26
        toks[k] = [word, b"%d" % k][k % 2] + [b")", b")+1", b"))"][k % 3]
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, pruning=False, walk_mode=0, state_cache_entries=-1)
    prefixes = [b"(a", b"a+b*c", b"((x", b"7*(a+b)"][:B]
    want, rows = [], []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
    for b in range(B):
        rows.append(eng.new_state())
        rows[-1].advance_bytes(prefixes[b % len(prefixes)])
    d_mask = torch.full((B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, rows, d_mask)
    report = eng.mask_report()
    assert report.walk_chunks > B * V // 30 and report.parser_steps > 0   # strings left to the parser; steps of the per-block automaton
    got = d_mask.cpu().numpy().view(np.uint32)
    for b in range(B):
        assert np.array_equal(got[b], want[b % len(prefixes)]), b


@pytest.mark.parametrize("V,B", [(33001, 200), (70001, 200), (33001, 256), (33001, 257), (2048, 2)])
def test_per_block_automaton_blocks_of_sixteen(V, B, torch_cuda, oracle_lib):
    """The same around the passes of a block of 16 wavefronts (1,024 words), with one block per row and with several, and at the batch from which on
    blocks are of 8 (256 compute units)."""
    test_per_block_automaton_passes(V, B, torch_cuda, oracle_lib)


@pytest.mark.parametrize("grammar,pruning,B", [("expr", False, 3), ("expr", False, 300), ("expr", True, 3), ("json", False, 3), ("json", True, 300)])
def test_per_block_automaton_terminals_that_go_on(grammar, pruning, B, torch_cuda, oracle_lib):
    """Runs of digits, letters and blanks, what ends them and what follows, from within a run and from its beginning, with charts of small and of large sets: the steps
    whose set is known from what Scan leaves, and those that are worked out before a string asks for them, against the oracle."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    if grammar == "expr":
        g, runs, joins, prefixes = configs.CONFIGS[5].grammar(), [b"1", b"12", b"777", b"a", b"ab"], [b"+", b"*", b")+", b"+(", b"*(", b")"], [b"", b"1", b"12", b"a+b*c+1", b"((x", b"1+2*3+4*5+6*7+8"]
    else:
        g, runs, joins, prefixes = grammars.json_grammar(), [b"1", b"12", b"7.25", b"  ", b"true"], [b",", b" ,", b"]", b"],", b":", b", "], [b"", b"[1", b"[12, 3", b'{"a": 1', b"[[ ", b'{"k" ']
    toks = runs + joins + [r + j + s for r in runs for j in joins for s in runs] + [r + j + r + j + r for r in runs for j in joins] + [r * 20 for r in runs] + [b""]
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, pruning=pruning, walk_mode=0, state_cache_entries=-1)
    want, rows = [], []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p), p
        want.append(so.mask(off, data, 8))
    for b in range(B):
        rows.append(eng.new_state())
        rows[-1].advance_bytes(prefixes[b % len(prefixes)])
    d_mask = torch.empty((B, eng.W), dtype=torch.int32, device="cuda")
    for at in ([0], [1], [2], list(range(3)), list(range(B))) if B <= 6 else (list(range(B)),):
        d_mask.fill_(0x5A5A5A5A)
        zf.compute_mask(eng, [rows[b] for b in at], d_mask[:len(at)])
        got = d_mask.cpu().numpy().view(np.uint32)
        for k, b in enumerate(at):
            assert np.array_equal(got[k], want[b % len(prefixes)]), (prefixes[b % len(prefixes)], len(at))


@pytest.mark.parametrize("words", [2, 1100], ids=["one pass", "passes"])
def test_per_block_automaton_drops_what_nobody_waits_for(words, torch_cuda, oracle_lib):
    """Sixty strings wait for the byte that they begin with, behind which none goes on: steps that were asked for ahead meanwhile, one for the second byte of each, are dropped
    when the strings are decided (with them a block took 61 steps).  In passes, transitions that were dropped are there for the strings of a later one."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    seconds = [bytes([c]) for c in range(140, 200)]
    g = grammars.Grammar("ahead").alts("S", [b"a", b"Z"], *[[c, b"Y"] for c in seconds], ["S", b"+", "S"]).set_start("S")   # (a grammar of operators: the step for a dozen items)
    toks = [b"a" + c for c in seconds] + [b""] * 4
    if words > 2:                                            # strings of other ranks: the last of them go the way of the steps that were dropped
        toks += [b"a" + bytes([100 + k % 30, 100 + k // 30 % 30, 100 + k // 900]) for k in range(32 * (words - 4))] + [c + e for c in seconds for e in (b"Y", b"Z")]
    off, data = wvocab.vocab_csr(toks)
    eng = zf.Engine(g, toks, device=0, walk_mode=0, token_mask_cache=False, state_cache_entries=-1)
    B = 1 if words == 2 else 300                              # 300 rows: a block each, of 512 words a pass
    want = oracle_lib.Oracle(g).new_state().mask(off, data, 8)
    d_mask = torch.full((B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    rows = [eng.new_state() for _ in range(B)]
    for _ in range(3):
        zf.compute_mask(eng, rows, d_mask)
        assert (d_mask.cpu().numpy().view(np.uint32) == want).all()
        assert 1 <= eng.mask_report().parser_steps < (50 if B == 1 else 250 * B)


@pytest.mark.parametrize("kw", [{}, {"walk_mode": 0}, {"pruning": False}], ids=["store", "per_block", "unpruned"])
def test_strings_that_a_terminal_may_end_in_everywhere(kw, torch_cuda, oracle_lib):
    """Cache rows made on the device: what follows every end that a terminal may have in a string is walked up to a number of bytes, with strings shorter and longer than that takes."""
    import paper_2506_01151_amd as zf
    from tests.test_host_library import dashes
    g, toks = dashes(2, [(b"a-" * k)[:2 * k - 1] + t + b"b" for k in (1, 2, 20, 21, 22, 23, 24, 30) for t in (b";", b"-", b")-", b"-;", b"(", b")")])
    orc, eng = oracle_lib.Oracle(g), zf.Engine(g, toks, device=0, state_cache_entries=-1, **kw)
    off, data = wvocab.vocab_csr(toks)
    want, rows = [], []
    for prefix in (b"", b"a", b"a-", b"a-a", b"(", b"(a", b"a;"):
        so = orc.new_state()
        rows.append(eng.new_state())
        if prefix:
            assert so.feed_bytes(prefix)
            rows[-1].advance_bytes(prefix)
        want.append(so.mask(off, data, 8))
    d_mask = torch_cuda.full((len(rows), eng.W), 0x5A5A5A5A, dtype=torch_cuda.int32, device="cuda")
    zf.compute_mask(eng, rows, d_mask)
    assert np.array_equal(d_mask.cpu().numpy().view(np.uint32), np.stack(want))


@pytest.mark.parametrize("depth", [40, 70, 120])
@pytest.mark.parametrize("pruning", [True, False], ids=["pruned", "unpruned"])
def test_per_block_automaton_steps_that_are_handed_over(depth, pruning, torch_cuda, oracle_lib):
    """A byte that completes `depth` rules at once and leaves 20 items: more than the step for a dozen items holds or tries (64, 96), so that the wide one takes it over, and
    what Scan had left is not known of the new set.  Item 20 of the set, before the completed ones are dropped, is a terminal that goes on in place, and the only one that
    the next byte leaves: with it for what Scan had left, that byte would lead back to the whole set."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    ends = [[b"m", "X", bytes([65 + k])] for k in range(19)]
    g = (grammars.Grammar("nest").alts("S", [b"q", "L"]).alts("L", [b"k", "L"], [b"k", "P"]).alts("P", *ends, [b"m", "X", grammars.Rx(rb"a*b")], [b"m", "X"])
         .alts("X", [b"x"]).set_start("S"))
    toks = [b"x", b"xa", b"xab", b"xaab", b"xb"] + [p + bytes([65 + k]) for k in range(19) for p in (b"x", b"xa", b"xaa", b"xab")] + [b"xaax", b"xx", b"", b"k", b"m"]
    prefix = b"q" + b"k" * depth + b"m"
    off, data = wvocab.vocab_csr(toks)
    so = oracle_lib.Oracle(g).new_state()
    assert so.feed_bytes(prefix)
    want = so.mask(off, data, 8)
    eng = zf.Engine(g, toks, device=0, pruning=pruning, walk_mode=0, token_mask_cache=False, state_cache_entries=-1)
    rows = [eng.new_state() for _ in range(3)]
    for r in rows:
        r.advance_bytes(prefix)
    for n in (1, 3):
        d_mask = torch.full((n, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        zf.compute_mask(eng, rows[:n], d_mask)
        assert eng.mask_report().parser_steps > 0 and eng.mask_report().overflow_chunks == 0
        for got in d_mask.cpu().numpy().view(np.uint32):
            assert np.array_equal(got, want), [t for k, t in enumerate(toks) if (got[k >> 5] ^ want[k >> 5]) >> (k & 31) & 1]


@pytest.mark.parametrize("V,B", [(16384, 300), (16385, 300), (33001, 200), (70001, 3), (33001, 257), (4097, 3), (2048, 2)])
@pytest.mark.parametrize("pruning", [True, False], ids=["pruned", "unpruned"])
def test_per_block_automaton_without_cache_rows(V, B, pruning, torch_cuda, oracle_lib):
    """Every string through the per-block automaton (no token-mask cache, so no row of it to ask for early), in one pass of a block and in several."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[5]
    g, toks = cfg.grammar(), cfg.vocab(V)
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, pruning=pruning, walk_mode=0, token_mask_cache=False, state_cache_entries=-1)
    prefixes = [b"", b"a+b*c", b"((x", b"7*(a+b)"][:B]
    want, rows = [], []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
    for b in range(B):
        rows.append(eng.new_state())
        rows[-1].advance_bytes(prefixes[b % len(prefixes)])
    d_mask = torch.full((B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, rows, d_mask)
    got = d_mask.cpu().numpy().view(np.uint32)
    for b in range(B):
        assert np.array_equal(got[b], want[b % len(prefixes)]), b


@pytest.mark.parametrize("n", [1, 7, 8, 9, 16, 63, 64, 65, 130])
def test_per_block_automaton_of_many_cache_rows(n, torch_cuda, oracle_lib):
    """Sets that select n rows of the token-mask cache (the words of up to 64 are asked for ahead of the chart, eight at a time), in passes with undecided strings
    and without: literals with a common beginning, a comma or a semicolon behind them by the context."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g = grammars.Grammar("many").alts("L", ["W", b",", "L"], [b"(", "M", b")"]).alts("M", ["W", b";", "M"], []).alts("W", *[[b"k%03d" % k] for k in range(n)]).set_start("L")
    toks = [b"", b"k", b"0", b"00", b"01", b"000", b"(", b",", b";"] + [b"%03d%s" % (k, e) for k in range(n + 2) for e in (b"", b",", b";", b",(", b";k", b";)", b",k0")]
    toks += [b"x%d" % k for k in range(40000)]                # passes of nothing but strings that are decided
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    prefixes = [b"k", b"(k", b"k0", b"(", b"(k000;k"]
    want = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p), p
        want.append(so.mask(off, data, 8))
    for pruning in (True, False):
        eng = zf.Engine(g, toks, device=0, pruning=pruning, walk_mode=0, state_cache_entries=-1)
        rows = [eng.new_state() for _ in prefixes]
        for r, p in zip(rows, prefixes):
            r.advance_bytes(p)
        for at in ([0], [1], list(range(len(prefixes)))):
            d_mask = torch.full((len(at), eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
            zf.compute_mask(eng, [rows[b] for b in at], d_mask)
            got = d_mask.cpu().numpy().view(np.uint32)
            for k, b in enumerate(at):
                assert np.array_equal(got[k], want[b]), (prefixes[b], pruning)


@pytest.mark.parametrize("n", [81800, 81919, 81920, 81921, 100003])
def test_closing_kernel_over_many_strings(n, torch_cuda, oracle_lib):
    """Rows of the rank-ordered bitmap of as many words as a block of the closing kernel requests at once, fewer and more, a last group of two rows: masks are
    the oracle's, logits masked along with them."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g = configs.CONFIGS[5].grammar()
    toks = [b"%d" % k for k in range(n - 60)] + [b"%d)+%d" % (k, k) for k in range(20)] + [b"%d+%d" % (k, k) for k in range(20)] + [b"%d)" % k for k in range(20)]
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, pruning=False, state_cache_entries=-1)
    prefixes = [b"", b"a+b*c", b"((x", b"7*(a+b)", b"(1"]
    want = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
    at = np.arange(50) % len(prefixes)
    rows = [eng.new_state() for _ in at]
    for r, p in zip(rows, at):
        r.advance_bytes(prefixes[p])
    logits = torch.randn((len(at), n), device="cuda")
    d_mask, out = torch.full((len(at), eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda"), torch.zeros_like(logits)
    zf.compute_mask_apply_async(eng, zf.StateBatch(rows), d_mask, logits, out=out)
    zf.mask_wait(eng)
    torch.cuda.synchronize()
    wanted = np.stack([want[p] for p in at])
    assert np.array_equal(d_mask.cpu().numpy().view(np.uint32), wanted)
    allowed = torch.from_numpy(np.unpackbits(wanted.view(np.uint8), axis=1, bitorder="little")[:, :n].astype(bool)).cuda()
    assert torch.equal(out, torch.where(allowed, logits, torch.full_like(logits, float("-inf"))))


@pytest.mark.parametrize("B,dtype", [(1, "f32"), (5, "bf16"), (70, "f32"), (300, "bf16")])
def test_calls_that_the_cache_rows_decide(B, dtype, torch_cuda, oracle_lib):
    """Without pruning: calls whose rows leave nothing to the parser (look-ups without any), of one group, of several and of more than the argument block holds, of more rows
    than it holds, of sentences that are complete, and calls of rows that leave something (the per-block automaton's) between them, with no wait but
    zf_mask_wait and on two streams; waiting calls; a state cache (which keeps to the per-block automaton).  Masks and logits are the oracle's."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g = grammars.Grammar("decided").alts("S", *[[b"k%03d" % k, b"!"] for k in range(90)], [b"(", "L", b")"]).alts("L", ["W", b",", "L"], ["W"], [b"[", "M", b"]"]).alts("M", ["W", b";", "M"], ["W"]).alts("W", [b"xy"], [b"xyz"]).set_start("S")
    toks = [b"", b"k", b"(", b"xy", b"xyz", b"y,", b"y;", b"y)", b"y,x", b"yz;xy", b"z", b"!", b"9!", b"(xy"] + [b"%02d" % k for k in range(100)] + [b"%03d!" % k for k in range(100)] + [b"n%d" % k for k in range(3000)]
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    decided = [b"k%03d" % k for k in range(90)] + [b"k", b"k0", b"", b"k001!", b"(xy,xyz)"]
    mixed = [b"(x", b"([x", b"(xy", b"([xyz"]
    masks = {}
    for p in decided + mixed:
        so = orc.new_state()
        assert not p or so.feed_bytes(p), p
        masks[p] = so.mask(off, data, 8)
    kind = torch.float32 if dtype == "f32" else torch.bfloat16
    V = len(toks)

    def batch(eng, prefixes):
        rows = [eng.new_state() for _ in prefixes]
        for r, p in zip(rows, prefixes):
            if p:
                r.advance_bytes(p)
        return zf.StateBatch(rows)

    eng = zf.Engine(g, toks, device=0, pruning=False, state_cache_entries=-1)
    lists = [[decided[k % len(decided)] for k in range(B)], [decided[-1]] * B, [mixed[k % len(mixed)] for k in range(B)], [(decided + mixed)[(7 * k) % (len(decided) + len(mixed))] for k in range(B)], [b"k"] * B, [decided[(3 * k) % 9] for k in range(B)]]
    batches = [batch(eng, x) for x in lists]
    order = [0, 0, 1, 4, 2, 0, 3, 5, 0, 2, 2, 4, 0, 1, 5, 3, 0, 0, 0]
    logits = torch.randn((len(order), B, V), device="cuda").to(kind)
    got = torch.full((len(order), B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    out = torch.zeros_like(logits)
    streams = [torch.cuda.current_stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for k, b in enumerate(order):
        with torch.cuda.stream(streams[1 if k in (8, 9, 10, 15) else 0]):
            zf.compute_mask_apply_async(eng, batches[b], got[k], logits[k], out=out[k])
            zf.mask_wait(eng)
    torch.cuda.synchronize()
    for k, b in enumerate(order):
        wanted = np.stack([masks[p] for p in lists[b]])
        assert np.array_equal(got[k].cpu().numpy().view(np.uint32), wanted), (k, b)
        allowed = torch.from_numpy(np.unpackbits(wanted.view(np.uint8), axis=1, bitorder="little")[:, :V].astype(bool)).cuda()
        assert torch.equal(out[k], torch.where(allowed, logits[k], torch.full_like(logits[k], float("-inf")))), (k, b)
    cached = zf.Engine(g, toks, device=0, pruning=False)
    for e in (eng, cached):
        for _ in range(2):
            for x in lists:
                one = torch.full((B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
                zf.compute_mask(e, batch(e, x), one)
                assert np.array_equal(one.cpu().numpy().view(np.uint32), np.stack([masks[p] for p in x]))


def test_host_diagnostics_of_an_engine_with_a_device(torch_cuda, oracle_lib):
    """The host's diagnostics read token-mask cache rows that an engine with a device does not hold on the host until somebody asks: each of them,
    the first to ask of an engine of its own."""
    import paper_2506_01151_amd as zf
    cfg = configs.CONFIGS[1]
    g, toks = cfg.grammar(), cfg.vocab()
    off, data = wvocab.vocab_csr(toks)
    so = oracle_lib.Oracle(g).new_state()
    assert so.feed_bytes(b'{"a": [1')
    want = so.mask(off, data)

    def twin(s):
        t = zf.binding.Twin(s.engine)
        rc, at, _ = t.advance(0, b'{"a": [1')
        assert rc == 0
        return t.mask(at)[0]

    for ask in (twin, lambda s: s.debug_host_mask_cached()[0], lambda s: s.debug_host_mask_automaton()[0]):
        s = zf.Engine(g, toks, device=0).new_state()
        s.advance_bytes(b'{"a": [1')
        assert np.array_equal(ask(s), want)


def test_host_diagnostics_asked_by_several_threads(torch_cuda, oracle_lib):
    """Eight threads ask an engine with a device for a host mask at once, the first anybody asks of it: one makes the rows, all have the oracle's mask."""
    import threading
    import paper_2506_01151_amd as zf
    cfg = configs.CONFIGS[2]
    g, toks = cfg.grammar(), cfg.vocab()
    off, data = wvocab.vocab_csr(toks)
    so = oracle_lib.Oracle(g).new_state()
    assert so.feed_bytes(b'{"a": [1')
    want = so.mask(off, data, 8)
    eng = zf.Engine(g, toks, device=0)
    rows, got, at_once = [eng.new_state() for _ in range(8)], [None] * 8, threading.Barrier(8)
    for s in rows:
        s.advance_bytes(b'{"a": [1')

    def ask(k):
        at_once.wait()
        got[k] = (rows[k].debug_host_mask_cached if k % 2 else rows[k].debug_host_mask_automaton)()[0]

    threads = [threading.Thread(target=ask, args=(k,)) for k in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(x is not None and np.array_equal(x, want) for x in got)


@pytest.mark.parametrize("walk_mode,pruning", [(0, True), (1, True), (2, False), (2, True)])
def test_first_call_on_a_stream_of_its_own(walk_mode, pruning, torch_cuda, oracle_lib):
    """The first mask call of an engine, right behind zf_compile and on a stream that does not wait for the null stream: strings and cache rows, which
    kernels on the null stream make, are there when zf_compile returns.  The masks are the oracle's."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g, toks = configs.CONFIGS[3].grammar(), configs.CONFIGS[3].vocab()
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    prefixes = [b"", b'{"']
    want = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
    side = torch.cuda.Stream()
    d_mask = torch.full((len(prefixes), (len(toks) + 31) // 32), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=walk_mode, pruning=pruning, precompute_states=-1)
    rows = [eng.new_state() for _ in prefixes]
    for s, p in zip(rows, prefixes):
        s.advance_bytes(p)
    with torch.cuda.stream(side):
        zf.compute_mask(eng, rows, d_mask)
    assert np.array_equal(d_mask.cpu().numpy().view(np.uint32), np.stack(want))


@pytest.mark.parametrize("V", [1, 31, 32, 33, 64, 65, 255, 256, 257, 2500])
@pytest.mark.parametrize("walk_mode", [0, 1, 2])
def test_token_mask_cache_made_on_the_device(V, walk_mode, torch_cuda, oracle_lib):
    """The rows of the token-mask cache and the strings' records as the device makes them -- vocabularies around a word, a wavefront and a block, tokens beyond the
    8, 15 and 16 bytes that are at hand and of the greatest length, empty ones among them -- against the host's walk of the trie with the host's rows."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    toks = [b'"' + b"k" * n for n in (0, 6, 7, 8, 13, 14, 15, 16, 40, 254)] + [b"", b"1" * 255, b'"a":', b"[[", b" ", b"-1.5e3"] + sorted(set(configs.CONFIGS[1].vocab(2048)))
    toks += [b"%d" % k for k in range(10, 2500)]
    toks = list(dict.fromkeys(toks))[:V][::-1]
    eng = zf.Engine(grammars.json_grammar(), toks, device=0, walk_mode=walk_mode, state_cache_entries=-1, precompute_states=-1)
    d_mask = torch.empty((1, eng.W), dtype=torch.int32, device="cuda")
    for prefix in (b"", b"[", b'{"x', b"[1", b'{"a": -', b"tr"):
        st = eng.new_state()
        st.advance_bytes(prefix)
        want, stats = st.debug_host_mask_cached()
        for call in range(2):
            zf.compute_mask(eng, [st], d_mask)
            assert np.array_equal(d_mask.cpu().numpy().view(np.uint32)[0], want), (prefix, call)
            if walk_mode == 2:
                assert eng.mask_report().walk_chunks == stats["undecided"], (prefix, call)   # no token twice: strings and tokens count the same


@pytest.mark.parametrize("token_cache", [True, False], ids=["", "parser-only"])
@pytest.mark.parametrize("pruning", [False, True])
@pytest.mark.parametrize("most", [2, 4, 5, 6, 7, 8, 12, 20, 40])
def test_byte_step_of_growing_sums(most, pruning, token_cache, torch_cuda, oracle_lib):
    """The per-block automaton's byte steps on sums of up to `most` operators of the ambiguous grammar, every operand another origin: sets from a few items, through the step
    for a dozen, to the wide one; origin sets and table entries to deal from fewer than the lanes of a wavefront to several times as many.  With the token-mask cache
    the strings that end a group are left to the parser, without it all."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[5]
    g = cfg.grammar()
    toks = list(dict.fromkeys(cfg.vocab(700) + [b"+b" * n for n in (1, 2, 5, 9)] + [b"*(" * 4, b")" * 3, b"+(a*b)" * 2, b"a" + b"+a" * 12]))
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, pruning=pruning, walk_mode=0, token_mask_cache=token_cache, state_cache_entries=-1)
    so, ss = [], []
    for k in range(most + 1):
        a, b = orc.new_state(), eng.new_state()
        p = b"(" * (k % 3) + b"a" + b"+b" * k + b"+" * (k % 2)
        assert a.feed_bytes(p)
        b.advance_bytes(p)
        so.append(a)
        ss.append(b)
    d_mask = torch.full((len(ss), eng.W), -1, dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, ss, d_mask)
    assert eng.mask_report().parser_steps > 0
    got = d_mask.cpu().numpy().view(np.uint32)
    for k, a in enumerate(so):
        assert (got[k] == a.mask(off, data, 4)).all(), k


def test_function_transforms_raise_and_the_process_goes_on(torch_cuda, oracle_lib):
    """The wrappers of vmap and grad pass for plain GPU tensors and refuse their address: an exception of Python's, and the next plain call is right."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    cfg = configs.CONFIGS[1]
    g, toks = cfg.grammar(), cfg.vocab()
    eng = zf.Engine(g, toks, device=0)
    st = eng.new_state()
    d_mask = torch.empty((1, eng.W), dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, [st], d_mask)
    logits = torch.randn((3, 1, eng.V), device="cuda")
    for f in (lambda: torch.func.vmap(lambda x: zf.apply_mask(eng, x, d_mask))(logits),
              lambda: torch.func.vmap(lambda x: zf.compute_mask_apply_async(eng, [st], d_mask, x))(logits),
              lambda: torch.func.grad(lambda x: zf.apply_mask(eng, x, d_mask).sum())(logits[0])):
        with pytest.raises(Exception):
            f()
    off, data = wvocab.vocab_csr(toks)
    want = oracle_lib.Oracle(g).new_state().mask(off, data)
    out = zf.apply_mask(eng, logits[0].clone(), zf.compute_mask(eng, [st], d_mask))
    assert out.cpu().numpy().view(np.uint32).tobytes() == oracle_apply(logits[0].cpu().numpy().view(np.uint32), want[None, :]).tobytes()


@pytest.mark.parametrize("noalloc,precompute", [(False, 0), (False, -1), (True, -1)])
def test_waiting_calls_on_two_streams(noalloc, precompute, torch_cuda, oracle_lib):
    """Waiting calls that take turns on two streams, nothing synchronised between them: the second call of a step is served the rows that the
    first has just left in the state cache (or walks the transitions it has just added), and the masks are the oracle's on both."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    cfg = configs.CONFIGS[4]
    g, toks = cfg.grammar(), cfg.vocab(16384)
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, precompute_states=precompute)
    call = zf.compute_mask_noalloc if noalloc else zf.compute_mask
    n, rs = 24, stream(11, f"two-streams{noalloc}{precompute}")
    first, second = [eng.new_state() for _ in range(n)], [eng.new_state() for _ in range(n)]
    oracles = [orc.new_state() for _ in range(n)]
    masks = [torch.full((n, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda") for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    hits = 0
    for step in range(10):
        for turn, rows in enumerate((first, second)):
            with torch.cuda.stream(streams[(step + turn) & 1]):
                call(eng, rows, masks[turn])
        hits += eng.mask_report().cache_hits
        got = [m.cpu().numpy().view(np.uint32) for m in masks]   # on the default stream, which waits for neither of the two
        for b in range(n):
            want = oracles[b].mask(off, data, 8)
            assert np.array_equal(got[0][b], want) and np.array_equal(got[1][b], want), (step, b)
            bits = np.flatnonzero(np.unpackbits(want.view(np.uint8), bitorder="little"))
            if len(bits) == 0:
                first[b].reset(), second[b].reset()
                oracles[b] = orc.new_state()
                continue
            t = int(bits[rs.below(len(bits))])
            first[b].advance(t), second[b].advance(t)
            assert oracles[b].feed_bytes(toks[t])
    assert noalloc or hits >= 9 * n, hits


@pytest.mark.parametrize("V,B,dtype,shift", [(5, 2, "f32", 0), (7, 1, "bf16", 1), (512, 3, "bf16", 0), (513, 70, "bf16", 0), (1023, 3, "f32", 3), (2047, 2, "bf16", 1), (2049, 66, "f32", 0),
                                             (8193, 5, "bf16", 5), (40037, 600, "bf16", 1), (33001, 300, "f32", 0)])
def test_logits_masked_along_with_look_ups(V, B, dtype, shift, torch_cuda, oracle_lib, polls=None):
    """The wavefronts of mask_look_kernel that mask logits: rows that end within a piece, within a KB and within a unit of four, rows at any multiple of
    an element, fewer tokens than a piece, groups in the argument block and beyond it, and tensors larger than what the chip holds at once (wavefronts that
    find their words there and leave out what nothing is allowed of).  Out of place; masks and logits are the oracle's."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    toks = (configs.CONFIGS[2].vocab(max(V, 2048))[::-1])[:V]
    off, data = wvocab.vocab_csr(toks)
    g = grammars.json_grammar()
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1)
    if polls is not None:
        zf.load_library().zf_debug_look_polls(eng.h, polls)
    prefixes = [b"", b"[", b'{"a', b"[1", b'["x', b"[[0.5e", b'{"k":', b"tru"] + [b"[" * k for k in range(2, 80 if B in (66, 70) else 2)]
    want = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
    rng = np.random.default_rng(V + B)
    u, i, f = (np.uint32, torch.int32, torch.float32) if dtype == "f32" else (np.uint16, torch.int16, torch.bfloat16)
    states = [eng.new_state() for _ in range(B)]
    rows = zf.StateBatch(states)
    wide = torch.zeros(B * (V + 3) + shift, dtype=i, device="cuda")
    d_mask, out = torch.empty((B, eng.W), dtype=torch.int32, device="cuda"), torch.empty(B * (V + 3) + shift, dtype=i, device="cuda")
    t, o = (x[shift:].view(B, V + 3)[:, :V] for x in (wide, out))
    for call in range(3):                          # the first call meets the states, the others look them up
        at = (np.arange(B) * 3 + 5 * call) % len(prefixes)
        for s, p in zip(states, at):
            s.reset()
            s.advance_bytes(prefixes[p])
        bits = rng.integers(0, np.iinfo(u).max, size=(B, V), dtype=u)
        t.copy_(torch.from_numpy(bits.view(np.int32 if dtype == "f32" else np.int16)))
        out.fill_(0x1234)
        zf.compute_mask_apply_async(eng, rows, d_mask, t.view(f), out=o.view(f))
        zf.mask_wait(eng)
        torch.cuda.synchronize()
        wanted = np.stack([want[p] for p in at])
        assert np.array_equal(d_mask.cpu().numpy().view(np.uint32), wanted), call
        assert np.ascontiguousarray(o.cpu().numpy()).view(u).tobytes() == oracle_apply(bits, wanted).tobytes(), call
        rest = out.cpu()
        rest[shift:].view(B, V + 3)[:, :V] = 0x1234
        assert bool((rest == 0x1234).all()), call   # nothing beyond the rows' ends


@pytest.mark.parametrize("V,B,dtype,shift", [(5, 2, "f32", 0), (513, 70, "bf16", 0), (2047, 2, "bf16", 1), (2049, 66, "f32", 0), (8193, 5, "bf16", 5), (40037, 600, "bf16", 1), (33001, 300, "f32", 0)])
def test_logits_left_to_the_block_that_is_last(V, B, dtype, shift, torch_cuda, oracle_lib):
    """The same with wavefronts that look for their mask words once: those that come before the words leave their logits to the block that is done last
    with the masks.  From one block of the mask to hundreds, records in the argument block and beyond it."""
    test_logits_masked_along_with_look_ups(V, B, dtype, shift, torch_cuda, oracle_lib, polls=0)


@pytest.mark.parametrize("V", [974848, 1048575])
def test_logits_masked_along_to_the_largest_grid(V, torch_cuda, oracle_lib):
    """4,096 rows of fp32 logits, 16 GB in place: about the most blocks that are counted in a group's 16 bits, and more than that (a launch of its own masks them)."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    B = 4096
    toks = (configs.CONFIGS[2].vocab(4096) + [b"%d" % k for k in range(10**7, 10**7 + V)])[:V]
    off, data = wvocab.vocab_csr(toks)
    g = grammars.json_grammar()
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1)
    prefixes, want, first = [b"[1", b'{"k":'], [], []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
        first.append(eng.new_state())
        first[-1].advance_bytes(p)
    rows = zf.StateBatch([first[b % 2].clone() for b in range(B)])
    base = torch.randn(V, device="cuda")
    logits = base.repeat(B, 1)
    d_mask = torch.full((B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, first, d_mask[:2])                  # the states have been met: what follows is look-ups
    zf.compute_mask_apply_async(eng, rows, d_mask, logits, out=logits)
    zf.mask_wait(eng)
    zf.mask_wait(eng)                                        # nothing in flight: for the calls that were let go of
    for k in range(2):
        allowed = torch.from_numpy(np.unpackbits(want[k].view(np.uint8), bitorder="little")[:V].astype(bool)).cuda()
        wanted, mask = torch.where(allowed, base, torch.full_like(base, float("-inf"))), torch.from_numpy(want[k].view(np.int32)).cuda()
        for b in range(k, B, 64):
            assert torch.equal(logits[b:b + 64:2], wanted.expand_as(logits[b:b + 64:2])), b
            assert torch.equal(d_mask[b:b + 64:2], mask.expand_as(d_mask[b:b + 64:2])), b


@pytest.mark.parametrize("polls", [None, 0, 3])
def test_look_ups_with_logits_of_two_engines_at_once(polls, torch_cuda, oracle_lib):
    """Two engines, each on a stream of its own, both with more blocks of logits than the chip holds: whichever blocks have the places, every logit is masked."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    V, B, calls = 64000, 96, 8
    toks = configs.CONFIGS[2].vocab(V)
    off, data = wvocab.vocab_csr(toks)
    g = grammars.json_grammar()
    orc = oracle_lib.Oracle(g)
    prefixes = [b"", b"[", b'{"a', b"[1", b'["x', b"[[0.5e", b'{"k":', b"tru"]
    want = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
    want = np.stack([want[b % 8] for b in range(B)])
    engines, rows = [zf.Engine(g, toks, device=0, state_cache_entries=-1) for _ in range(2)], []
    for e in engines:
        if polls is not None:
            zf.load_library().zf_debug_look_polls(e.h, polls)
        batch = [e.new_state() for _ in range(B)]
        for b, s in enumerate(batch):
            s.advance_bytes(prefixes[b % 8])
        rows.append(zf.StateBatch(batch))
    streams = [torch.cuda.Stream() for _ in engines]
    logits = torch.randn(B, V, device="cuda")
    masks = torch.full((2, calls, B, engines[0].W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    outs = torch.zeros((2, calls, B, V), device="cuda")
    torch.cuda.synchronize()
    for call in range(calls):                      # the first call meets the states
        for k, e in enumerate(engines):
            with torch.cuda.stream(streams[k]):
                zf.compute_mask_apply_async(e, rows[k], masks[k, call], logits, out=outs[k, call])
                zf.mask_wait(e)
    torch.cuda.synchronize()
    allowed = torch.from_numpy(np.unpackbits(want.view(np.uint8), axis=1, bitorder="little")[:, :V].astype(bool)).cuda()
    wanted = torch.where(allowed, logits, torch.full_like(logits, float("-inf")))
    for k in range(2):
        for call in range(calls):
            assert np.array_equal(masks[k, call].cpu().numpy().view(np.uint32), want), (k, call)
            assert torch.equal(outs[k, call], wanted), (k, call)


@pytest.mark.parametrize("dtype,shift", [("f32", 0), ("bf16", 1)])
@pytest.mark.parametrize("walk_mode,V,B", [(0, 1, 1), (0, 3, 2), (1, 31, 3), (0, 33, 4), (0, 255, 5), (1, 257, 6), (0, 1023, 9), (0, 1026, 64), (0, 2053, 130), (1, 8195, 70),
                                           (0, 8195, 601), (0, 40037, 110)])
def test_logits_masked_along_by_the_closing_kernel(walk_mode, V, B, dtype, shift, torch_cuda, oracle_lib):
    """finish_kernel with logits and without: vocabularies that end within a lane's four tokens, a word, a wavefront's 256 and a block's pass, batches that
    end within a group of four rows, rows at any multiple of an element, the rows in LDS (from 8,195 x 601 on) and groups of rows in turn.
    Masks and logits are the oracle's, with nothing stored beyond the rows' ends."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    toks = (configs.CONFIGS[2].vocab(max(V, 2048))[::-1])[:V]
    off, data = wvocab.vocab_csr(toks)
    g = grammars.json_grammar()
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, walk_mode=walk_mode, state_cache_entries=-1)
    prefixes = [b"", b"[", b'{"a', b"[1", b'["x', b'{"k":', b"tru"]
    want = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
    at = np.arange(B) * 3 % len(prefixes)
    wanted = np.stack([want[p] for p in at])
    states = [eng.new_state() for _ in range(B)]
    for s, p in zip(states, at):
        s.advance_bytes(prefixes[p])
    rows = zf.StateBatch(states)
    u, i, f = (np.uint32, torch.int32, torch.float32) if dtype == "f32" else (np.uint16, torch.int16, torch.bfloat16)
    bits = np.random.default_rng(V + B).integers(0, np.iinfo(u).max, size=(B, V), dtype=u)
    wide = torch.zeros(B * (V + 3) + shift, dtype=i, device="cuda")
    guard = torch.full((B + 2, eng.W), 0x1234, dtype=torch.int32, device="cuda")
    out = torch.full((B * (V + 3) + shift,), 0x1234, dtype=i, device="cuda")
    t, o = (x[shift:].view(B, V + 3)[:, :V] for x in (wide, out))
    t.copy_(torch.from_numpy(bits.view(np.int32 if dtype == "f32" else np.int16)))
    zf.compute_mask_apply_async(eng, rows, guard[1:-1], t.view(f), out=o.view(f))
    zf.mask_wait(eng)
    torch.cuda.synchronize()
    assert np.array_equal(guard[1:-1].cpu().numpy().view(np.uint32), wanted)
    assert np.ascontiguousarray(o.cpu().numpy()).view(u).tobytes() == oracle_apply(bits, wanted).tobytes()
    rest = out.cpu()
    rest[shift:].view(B, V + 3)[:, :V] = 0x1234
    assert bool((rest == 0x1234).all()) and bool((guard[0] == 0x1234).all()) and bool((guard[-1] == 0x1234).all())
    guard.fill_(0x77)
    zf.compute_mask(eng, rows, guard[1:-1])
    assert np.array_equal(guard[1:-1].cpu().numpy().view(np.uint32), wanted)


@pytest.mark.parametrize("B", [1, 5, 252, 300])
@pytest.mark.parametrize("n", [1, 8, 9, 10, 11, 12, 13, 16, 72, 73, 140, 255, 256])
def test_look_ups_of_states_with_many_cache_rows(n, B, torch_cuda, oracle_lib):
    """mask_look_kernel on states whose `n` items each have a token-mask cache row of their own (n terminals have one byte in common): around the nine rows a record
    holds, around the four that are read and the 64 that are numbered at a time, the most the short form counts and one more (the other kernel's); rows and members in the argument
    block together and apart.  The second call is the one of look-ups."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    g = grammars.Grammar(name=f"one_byte_in_common_{n}")
    g.set_start("S")
    words = [b"a%03d" % k + bytes([97 + k % 26]) * (k % 5) for k in range(n)]
    for w in words:
        g.rule("S", [w, "E"])
    g.rule("E", [b"!"])
    toks = list(dict.fromkeys([b"a", b"!", b"0", b"00", b"01", b"1", b"12", b"25", b"b!", b"bb", b"a0"] + [w[1:] for w in words] + [w[1:] + b"!" for w in words[::3]] + [b"%03d" % k for k in range(0, 300, 7)] + [b"zz%d" % k for k in range(700)]))
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1)
    prefixes = [b"a", b"a0", b"", b"a"]
    want = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 4))
    at = np.arange(B) % len(prefixes)
    wanted = np.stack([want[p] for p in at])
    states = [eng.new_state() for _ in range(B)]
    for s, p in zip(states, at):
        s.advance_bytes(prefixes[p])
    rows = zf.StateBatch(states)
    bits = np.random.default_rng(n + B).integers(0, 2**32, size=(B, eng.V), dtype=np.uint32)
    t = torch.from_numpy(bits.view(np.int32)).cuda()
    d_mask, out = torch.empty((B, eng.W), dtype=torch.int32, device="cuda"), torch.empty_like(t)
    for call in range(3):
        d_mask.fill_(-1); out.fill_(7)
        zf.compute_mask_apply_async(eng, rows, d_mask, t.view(torch.float32), out=out.view(torch.float32))
        zf.mask_wait(eng)
        torch.cuda.synchronize()
        assert np.array_equal(d_mask.cpu().numpy().view(np.uint32), wanted), call
        assert out.cpu().numpy().view(np.uint32).tobytes() == oracle_apply(bits, wanted).tobytes(), call


@pytest.mark.parametrize("B,dtype", [(3, "bf16"), (64, "f32"), (300, "bf16")])
def test_calls_that_mask_wait_lets_go_of(B, dtype, torch_cuda, oracle_lib):
    """Calls of look-ups only, one behind the other with nothing synchronised between them: more of them than there are slots, records and row numbers
    in the slots' own memory (300 rows), a change of streams with calls still at work, the store filled anew behind them, and a waiting call.
    Every step's mask and masked logits are the oracle's."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    cfg = configs.CONFIGS[3]
    g, toks, V, steps = cfg.grammar(), cfg.vocab(8192), 8192, 18
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1)      # no recursion: the automaton is there whole, every call is of look-ups only
    run = OracleRun(oracle_lib.Oracle(g), toks, [stream(31, f"let-go[{k}]") for k in range(8)])
    rows = zf.StateBatch([eng.new_state() for _ in range(B)])
    u, i, f = (np.uint32, torch.int32, torch.float32) if dtype == "f32" else (np.uint16, torch.int16, torch.bfloat16)
    rng = np.random.default_rng(B)
    bits = rng.integers(0, np.iinfo(u).max, size=(B, V), dtype=u)
    logits = torch.from_numpy(bits.view(np.int32 if dtype == "f32" else np.int16)).cuda().view(f)
    masks = torch.full((steps, B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    outs = torch.zeros((steps, B, V), dtype=f, device="cuda")
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    want = []
    for step in range(steps):
        want.append(run.masks())
        ids = run.step(want[-1])
        if step in (9, 14):
            eng.clear_state_cache()
        with torch.cuda.stream(streams[step // 6 & 1]):
            if step == 16:
                zf.compute_mask(eng, rows, masks[step])
                zf.apply_mask(eng, logits, masks[step], out=outs[step])
            else:
                zf.compute_mask_apply_async(eng, rows, masks[step], logits, out=outs[step])
                zf.mask_wait(eng)
        rows.advance([ids[b % 8] for b in range(B)])
    torch.cuda.synchronize()
    for step in range(steps):
        wanted = np.stack([want[step][b % 8] for b in range(B)])
        assert np.array_equal(masks[step].cpu().numpy().view(np.uint32), wanted), step
        assert outs[step].view(i).cpu().numpy().view(u).tobytes() == oracle_apply(bits, wanted).tobytes(), step


def test_failures_of_calls_that_mask_wait_has_let_go_of(torch_cuda, oracle_lib):
    """A call of look-ups that reports failed walks after mask_wait has let go of it: mask_wait with nothing in flight says so, and so does a waiting call,
    whose own mask is right, and which is not taken for the one that failed (nothing is answered again, the persistent automaton is not put on hold).  A waiting
    call's own failure is answered again; a call that leaves rows in the state cache is not let go of."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g, toks = configs.CONFIGS[3].grammar(), configs.CONFIGS[3].vocab(8192)
    off, data = wvocab.vocab_csr(toks)
    so = oracle_lib.Oracle(g).new_state()
    assert so.feed_bytes(b'{"')
    want = so.mask(off, data, 8)
    lib, logits = zf.load_library(), torch.randn(1, len(toks), device="cuda")

    def engine(**kw):
        eng = zf.Engine(g, toks, device=0, **kw)         # no recursion: every call is of look-ups only
        rows = zf.StateBatch([eng.new_state()])
        rows.states[0].advance_bytes(b'{"')
        return eng, rows, torch.full((1, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")

    def good(d_mask):
        torch.cuda.synchronize()
        return np.array_equal(d_mask.cpu().numpy().view(np.uint32)[0], want)

    def start(eng, rows, d_mask, apply, failing=3):
        assert lib.zf_debug_fail_look_ups(eng.h, failing) == 0
        if apply:
            zf.compute_mask_apply_async(eng, rows, d_mask, logits)
        else:
            zf.compute_mask_async(eng, rows, d_mask)

    for apply in (False, True):
        eng, rows, d_mask = engine(state_cache_entries=-1)
        start(eng, rows, d_mask, apply)
        zf.mask_wait(eng)                                # let go of
        with pytest.raises(zf.ZfError, match="3 walks failed in a call of look-ups that zf_mask_wait had let go of"):
            zf.mask_wait(eng)                            # nothing in flight
        zf.mask_wait(eng)                                # said once
        zf.compute_mask(eng, rows, d_mask)
        assert good(d_mask)
        start(eng, rows, d_mask, apply)
        zf.mask_wait(eng)
        other = torch.full_like(d_mask, 0x5A5A5A5A)
        with pytest.raises(zf.ZfError, match="let go of"):
            zf.compute_mask(eng, rows, other)
        assert good(other)
        eng.set_profiling(True)
        zf.compute_mask(eng, rows, d_mask)
        assert eng.mask_report().permute_ms == 0 and good(d_mask)   # no closing kernel: not through the per-block automaton
        eng.set_profiling(False)
    zf.compute_mask(eng, rows, d_mask)
    lib.zf_debug_fail_look_ups(eng.h, 5)
    d_mask.fill_(-1)
    eng.set_profiling(True)
    zf.compute_mask(eng, rows, d_mask)                   # its own failure: answered through the per-block automaton
    assert good(d_mask) and eng.mask_report().permute_ms > 0
    eng, rows, d_mask = engine()                         # the state cache on
    start(eng, rows, d_mask, False)
    with pytest.raises(zf.ZfError, match="exceeded the fallback arena"):
        zf.mask_wait(eng)


@pytest.mark.parametrize("walk_mode,pruning", [(0, True), (1, True), (2, False)])
def test_status_ahead_of_the_closing_kernel_and_another_stream(walk_mode, pruning, torch_cuda, oracle_lib):
    """mask_wait returns when a call's closing kernel has begun; the next call comes on another stream, nothing synchronised between them, and does not
    write the verdicts that the first kernel still reads.  Rows stand in other states from call to call; masks and masked logits are the oracle's."""
    import paper_2506_01151_amd as zf
    from oracle.frontend import apply_mask as oracle_apply
    torch = torch_cuda
    g, toks, B, calls = configs.CONFIGS[2].grammar(), configs.CONFIGS[2].vocab(32000), 64, 12
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=walk_mode, pruning=pruning)
    prefixes = [b"", b'{"a": [1', b'{"', b"[[", b'{"a": tr']
    per_state, rows = [], []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        per_state.append(so.mask(off, data, 8))
        rows.append([eng.new_state() for _ in range(B)])
        for s in rows[-1]:
            s.advance_bytes(p)
    logits = torch.randn(B, len(toks), device="cuda")
    masks = torch.full((calls, B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    outs = torch.zeros((calls, B, len(toks)), device="cuda")
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    for call in range(calls):
        with torch.cuda.stream(streams[call % 3]):
            zf.compute_mask_apply_async(eng, [rows[(b + call) % len(rows)][b] for b in range(B)], masks[call], logits, out=outs[call])
            zf.mask_wait(eng)
    torch.cuda.synchronize()
    bits = logits.cpu().numpy().view(np.uint32)
    for call in range(calls):
        want = np.stack([per_state[(b + call) % len(rows)] for b in range(B)])
        assert np.array_equal(masks[call].cpu().numpy().view(np.uint32), want), call
        assert outs[call].cpu().numpy().view(np.uint32).tobytes() == oracle_apply(bits, want).tobytes(), call


@pytest.mark.parametrize("walk_mode", [0, 2])
def test_threads_that_take_turns_on_their_own_streams(walk_mode, torch_cuda, oracle_lib):
    """Two threads that take turns with an engine, each on its per-thread default stream -- one handle, two streams: a call goes behind the one before it.  More
    calls than slots, rows in other states each time; masks and masked logits are the oracle's."""
    import threading
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g, toks, B, calls = configs.CONFIGS[3].grammar(), configs.CONFIGS[3].vocab(8192), 96, 12
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=walk_mode)
    prefixes, per_state, rows = [b"", b"{", b'{"'], [], []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        per_state.append(so.mask(off, data, 8))
        rows.append([eng.new_state() for _ in range(B)])
        for s in rows[-1]:
            s.advance_bytes(p)
    logits = torch.randn(B, len(toks), device="cuda")
    masks = torch.full((calls, B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    outs = torch.zeros((calls, B, len(toks)), device="cuda")
    torch.cuda.synchronize()
    turn, failed = [threading.Semaphore(1), threading.Semaphore(0)], []

    def work(k):
        for call in range(k, calls, 2):
            turn[k].acquire()
            try:
                with torch.cuda.stream(torch.cuda.ExternalStream(2)):   # hipStreamPerThread
                    zf.compute_mask_apply_async(eng, [rows[(b + call) % 3][b] for b in range(B)], masks[call], logits, out=outs[call])
                    zf.mask_wait(eng)
            except Exception as e:
                failed.append(e)
            turn[1 - k].release()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
    torch.cuda.synchronize()
    for call in range(calls):
        want = np.stack([per_state[(b + call) % 3] for b in range(B)])
        allowed = torch.from_numpy(np.unpackbits(want.view(np.uint8), axis=1, bitorder="little")[:, :len(toks)].astype(bool)).cuda()
        assert np.array_equal(masks[call].cpu().numpy().view(np.uint32), want), call
        assert torch.equal(outs[call], torch.where(allowed, logits, torch.full_like(logits, float("-inf")))), call


def test_look_ups_behind_a_per_block_call_in_flight(torch_cuda, oracle_lib):
    """A call of look-ups right behind one through the per-block automaton, both in flight: mask_wait has the status of the first as well (the report
    counts what its item budget of two left to the fallback pass), and calls that use its slot again find it free.  Masks are the oracle's."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g, toks, B = configs.CONFIGS[3].grammar(), configs.CONFIGS[3].vocab(8192), 64
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, lane_item_cap=2)
    prefixes = [b"", b"{", b'{"']
    want = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
    want = np.stack([want[b % 3] for b in range(B)])
    rows = [eng.new_state() for _ in range(B)]
    for b, s in enumerate(rows):
        s.advance_bytes(prefixes[b % 3])
    masks = torch.full((15, B, eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")

    def check(k):
        assert np.array_equal(masks[k].cpu().numpy().view(np.uint32), want), k

    zf.compute_mask_async(eng, rows, masks[0])
    eng.clear_state_cache()                        # with a call in flight: the store starts empty, and sets outgrow the budget
    zf.mask_wait(eng)
    zf.compute_mask(eng, rows, masks[1])           # does not fit the store: the next eight calls take the per-block automaton
    check(0), check(1)
    eng.clear_state_cache()                        # the automaton whole again
    for k in range(7):
        zf.compute_mask_async(eng, rows, masks[2 + k])
        zf.mask_wait(eng)
        assert eng.mask_report().overflow_chunks > 0, k
    zf.compute_mask_async(eng, rows, masks[9])     # the eighth
    zf.compute_mask_async(eng, rows, masks[10])    # look-ups
    zf.mask_wait(eng)
    assert eng.mask_report().overflow_chunks > 0   # of the eighth: its status was there
    for k in range(11, 15):
        zf.compute_mask_async(eng, rows, masks[k])
        zf.mask_wait(eng)
        assert eng.mask_report().overflow_chunks == 0, k
    for k in range(2, 15):
        check(k)


@pytest.mark.parametrize("walk_mode,noalloc", [(0, False), (1, False), (0, True)])
def test_fallback_passes_of_two_engines_at_once(walk_mode, noalloc, torch_cuda, oracle_lib):
    """Two engines, each on a stream of its own, whose strings all go to the fallback pass: their closing kernels share the chip, and neither waits for
    blocks of its own that have no place.  (The call that allocates nothing has fewer arenas than blocks; its calls take turns.)  Masks are the oracle's."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g, toks, B = configs.CONFIGS[3].grammar(), configs.CONFIGS[3].vocab(8192), 24 if noalloc else 130
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    prefixes = [b"", b"{", b'{"']
    want = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data, 8))
    want = np.stack([want[b % 3] for b in range(B)])
    engines = [zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=walk_mode, lane_item_cap=1) for _ in range(2)]
    rows = [[e.new_state() for _ in range(B)] for e in engines]
    for batch in rows:
        for b, s in enumerate(batch):
            s.advance_bytes(prefixes[b % 3])
    streams = [torch.cuda.Stream() for _ in engines]
    masks = torch.full((2, 4, B, engines[0].W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for call in range(4):
        for k, e in enumerate(engines):
            with torch.cuda.stream(streams[k]):
                (zf.compute_mask_noalloc if noalloc else zf.compute_mask_async)(e, rows[k], masks[k, call])
    for k, e in enumerate(engines):
        with torch.cuda.stream(streams[k]):
            zf.mask_wait(e)
        assert e.mask_report().overflow_chunks > 0
    torch.cuda.synchronize()
    got = masks.cpu().numpy().view(np.uint32)
    for k in range(2):
        for call in range(4):
            assert np.array_equal(got[k, call], want), (k, call)


def test_per_block_automaton_sets_that_outgrow_the_lanes(torch_cuda, oracle_lib):
    """Charts whose sets hold ten items, and a byte that leaves eighty: more than the build for a dozen items holds.  The call that allocates
    nothing does not take that build (nothing is left to the fallback pass); another call leaves the strings behind the byte to that pass once, and
    the engine's next calls take the build that holds the set.  Masks are the oracle's throughout."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    from workloads.grammar import Grammar
    g = Grammar(name="keywords")
    g.set_start("S")
    g.alts("S", *[[f"A{k}", "K", f"A{k}"] for k in range(10)])
    for k in range(10):
        g.alts(f"A{k}", [b"a"])
    words = [b"k%02dx" % k for k in range(80)]
    g.alts("K", *[[w] for w in words])
    toks = [bytes([c]) for c in range(128)] + words + [b"k0", b"k1", b"k07xa", b"k79xb", b"ak33xa", b"aa", b"k80x"] + [b"k%dx" % k for k in range(40)]
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    want = []
    for p in (b"", b"a", b"ak", b"ak4", b"ak42x"):
        so = orc.new_state()
        assert so.feed_bytes(p)
        want.append(so.mask(off, data))
    engines = [zf.Engine(g, toks, device=0, state_cache_entries=-1, walk_mode=0) for _ in range(2)]
    d_mask = torch.empty((2, engines[0].W), dtype=torch.int32, device="cuda")

    def masks(eng, call, prefixes):
        rows = []
        for p in prefixes:
            rows.append(eng.new_state())
            rows[-1].advance_bytes(p)
        d_mask.fill_(0x5A5A5A5A)
        call(eng, rows, d_mask)
        return d_mask.cpu().numpy().view(np.uint32), eng.mask_report().overflow_chunks

    start = engines[0].new_state()
    start.advance_bytes(b"a")
    assert sum(1 for it in start.chart()[0] if it[0] == 1) == 10     # the current set: more than the narrow build takes, no more than the next one
    got, left = masks(engines[0], zf.compute_mask_noalloc, (b"", b"a"))
    assert np.array_equal(got, np.stack(want[:2])) and left == 0
    for turn in range(3):
        got, left = masks(engines[1], zf.compute_mask, (b"", b"a"))
        assert np.array_equal(got, np.stack(want[:2])) and (left > 0) == (turn == 0), (turn, left)
    for k, p in ((2, b"ak"), (3, b"ak4"), (4, b"ak42x")):
        got, left = masks(engines[1], zf.compute_mask, (b"a", p))
        assert np.array_equal(got, np.stack([want[1], want[k]])), p


def test_advance_goes_on_while_the_automaton_is_explored_again(torch_cuda, oracle_lib):
    """zf_engine_clear_state_cache explores the automaton again (of this ambiguous grammar for tens of milliseconds); a row that another thread
    feeds meanwhile waits for a transition now and then, not for the exploration, and its mask is the oracle's afterwards."""
    import threading
    import time
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    from workloads.grammar import Grammar
    g = Grammar(name="ambiguous")
    g.set_start("S")
    g.alts("S", ["S", "S"], ["S", "S", "S"], ["S", b"+", "S"], [b"(", "S", b")"], [b"a"], [b"b"])
    toks = [bytes([c]) for c in range(128)] + [b"ab", b"a+", b"(a", b"aaa", b"b)", b")b"]
    off, data = wvocab.vocab_csr(toks)
    so = oracle_lib.Oracle(g).new_state()
    text = b"(a+b)ab(a" * 3
    assert so.feed_bytes(text)
    eng = zf.Engine(g, toks, device=0, state_cache_entries=-1)
    row = eng.new_state()
    for attempt in range(4):                             # (a thread that the machine takes off its core for a moment is no fault of the lock)
        took, longest, n, done = [], 0.0, 0, threading.Event()

        def clear():
            t = time.perf_counter()
            eng.clear_state_cache()
            took.append(time.perf_counter() - t)
            done.set()

        thread = threading.Thread(target=clear)
        thread.start()
        while not done.is_set():
            row.reset()
            for c in text:
                t = time.perf_counter()
                row.advance(c)
                longest = max(longest, time.perf_counter() - t)
                n += 1
        thread.join()
        print(f"cleared in {took[0] * 1e3:.0f} ms, {n} advances meanwhile, the longest {longest * 1e3:.1f} ms")
        if longest < 0.5 * took[0]:
            break
    else:
        raise AssertionError((took[0], longest))
    row.reset()
    for c in text:
        row.advance(c)
    d_mask = torch.empty((1, eng.W), dtype=torch.int32, device="cuda")
    zf.compute_mask(eng, [row], d_mask)
    assert np.array_equal(d_mask.cpu().numpy().view(np.uint32)[0], so.mask(off, data))


@pytest.mark.parametrize("V", [1, 33, 5000])
def test_vocabulary_of_empty_tokens(V, torch_cuda):
    """No string at all: every mask word is zero and every logit -inf, through the waiting, the asynchronous and the allocation-free call, on every path."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    for kw in ({}, {"state_cache_entries": -1, "precompute_states": -1}, {"walk_mode": 0}, {"walk_mode": 1}, {"pruning": False}):
        eng = zf.Engine(grammars.json_grammar(), [b""] * V, device=0, **kw)
        rows = []
        for p in (b"", b"[", b'{"k":"', b"[1,", b'[[{"a":[', b"[]"):
            rows.append(eng.new_state())
            if p:
                rows[-1].advance_bytes(p)
        d_mask = torch.empty((len(rows), eng.W), dtype=torch.int32, device="cuda")
        logits = torch.ones((len(rows), V), device="cuda")
        for call in (zf.compute_mask, zf.compute_mask_noalloc, zf.compute_mask_async):
            d_mask.fill_(0x5A5A5A5A)
            call(eng, rows, d_mask)
            zf.mask_wait(eng)
            torch.cuda.synchronize()
            assert not d_mask.any(), (kw, call)
        out = zf.compute_mask_apply_async(eng, rows, d_mask, logits, out=torch.empty_like(logits))
        zf.mask_wait(eng)
        torch.cuda.synchronize()
        assert not d_mask.any() and bool((out == float("-inf")).all()), kw


@pytest.mark.parametrize("V,B,pad,dtype", [(40000, 640, 0, "bf16"), (40003, 641, 61, "bf16"), (128256, 197, 0, "bf16"), (40000, 321, 64, "f32"), (12582, 1001, 2, "f32")])
def test_apply_mask_large_tensors_skip_empty_pieces(V, B, pad, dtype, torch_cuda, oracle_lib):
    """Aligned rows beyond the size from which pieces that nothing is allowed of are not read: whole words and whole rows empty and full, in
    place and into another tensor, every bit against the definition."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    from oracle.frontend import apply_mask as oracle_apply
    f, i, u = (torch.float32, torch.int32, np.uint32) if dtype == "f32" else (torch.bfloat16, torch.int16, np.uint16)
    assert (V // (4 if dtype == "f32" else 8)) * B >= 3 << 20 and (V + pad) * (4 if dtype == "f32" else 2) % 16 == 0
    eng = zf.Engine(grammars.parens_grammar(), [b"("] * V, device=0)
    rng = np.random.default_rng(V + B)
    mask = rng.integers(0, 2**32, size=(B, eng.W), dtype=np.uint32) & rng.integers(0, 2**32, size=(B, eng.W), dtype=np.uint32)
    mask[rng.random((B, eng.W)) < 0.4] = 0
    mask[0] = 0
    mask[-1] = 0xFFFFFFFF
    mask[B // 2] = 0
    bits = rng.integers(0, np.iinfo(u).max, size=(B, V), dtype=u)
    want = oracle_apply(bits, mask)
    x = torch.zeros((B, V + pad), dtype=f, device="cuda")[:, :V]
    x.view(i).copy_(torch.from_numpy(bits.view(np.int32 if dtype == "f32" else np.int16)))
    m = torch.from_numpy(mask.view(np.int32)).cuda()
    out = torch.empty_strided(x.shape, x.stride(), dtype=f, device="cuda")
    for y in (zf.apply_mask(eng, x, m, out=out), zf.apply_mask(eng, x, m)):
        assert y.contiguous().view(i).cpu().numpy().view(u).tobytes() == want.tobytes()


def _many_states():
    """A grammar of 2,600 words told apart by their first four bytes, in twenty terminals: as many states of one item each; what may follow is the word's fifth byte."""
    from workloads.grammar import Grammar, Rx
    g = Grammar(name="words")
    g.set_start("S")
    stems = [b"%04x" % (7 * k) for k in range(2600)]
    ends = [bytes([ord("g") + k % 20]) for k in range(2600)]
    words = [s + e + s for s, e in zip(stems, ends)]         # (the stem again: no two words share a state of their terminal's machine)
    g.alts("S", *[[Rx(b"(" + b"|".join(words[j::20]) + b")")] for j in range(20)])
    toks = [bytes([c]) for c in range(128)] + [b"g" * 2, b"z", b"h", b""] + [b"%xk" % k for k in range(16)]
    want = np.zeros((2600, (len(toks) + 31) // 32), dtype=np.uint32)
    for k, e in enumerate(ends):
        for t, tok in enumerate(toks):
            if tok == e:
                want[k, t >> 5] |= np.uint32(1 << (t & 31))
    return g, toks, stems, want


def test_calls_of_many_groups(torch_cuda, oracle_lib):
    """Calls of hundreds and thousands of groups, whose records travel in device memory: through the call that allocates nothing (records in the static
    array) up to the call whose records no longer fit its staging room, which goes to the per-block automaton; and with the state cache on, where some
    groups' masks are in the pool and others' are not."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g, toks, stems, want = _many_states()
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    for k in (0, 1, 19, 2599):                               # the table above, as the oracle sees it
        so = orc.new_state()
        assert so.feed_bytes(stems[k])
        assert np.array_equal(so.mask(off, data), want[k])

    def rows_of(eng, ks):
        rows = []
        for k in ks:
            rows.append(eng.new_state())
            rows[-1].advance_bytes(stems[k])
        return rows

    def check(eng, call, rows, ks, turn):
        d_mask = torch.full((len(ks), eng.W), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        call(eng, rows, d_mask)
        if call is zf.compute_mask_async:
            zf.mask_wait(eng)
        got = d_mask.cpu().numpy().view(np.uint32)
        assert np.array_equal(got, want[ks]), (len(ks), turn, np.flatnonzero((got != want[ks]).any(axis=1))[:8])
        return eng.mask_report()

    for precompute in (0, -1):                               # explored to its end: look-ups; not explored: first visits, then look-ups
        eng = zf.Engine(g, toks, device=0, state_cache_entries=-1, precompute_states=precompute)
        rows = rows_of(eng, range(2600))
        for n in (65, 300, 2000, 2600, 300):
            ks = [(3 * k + n) % 2600 for k in range(n)] if n < 2600 else list(range(2600))
            for turn in range(2):
                r = check(eng, zf.compute_mask_noalloc, [rows[k] for k in ks], ks, turn)
                assert r.chart_bytes <= 256 << 10, (n, turn, r.chart_bytes)   # 2,600 groups' records and blocks take 280 KiB: the packed charts went instead
                if precompute == 0 or turn == 1:
                    assert r.parser_steps == 0, (n, turn, r.parser_steps)
    eng = zf.Engine(g, toks, device=0)                       # the state cache at its default: 2,048 rows
    rows = rows_of(eng, range(2600))
    seen = set()
    for call in (zf.compute_mask, zf.compute_mask_async):
        for lo, hi in ((0, 100), (50, 250), (0, 300), (299, 301), (200, 1000)):
            ks = list(range(lo, hi))
            r = check(eng, call, [rows[k] for k in ks], ks, 0)
            assert r.cache_hits == len(seen & set(ks)) and r.cache_misses == len(ks) - r.cache_hits, (lo, hi, r.cache_hits)
            seen |= set(ks)


def test_state_cache_when_the_host_automaton_starts_over(torch_cuda, oracle_lib):
    """The cached masks go by the host automaton's names: when that fills up and starts over -- here a row of another query is fed sixty thousand
    brackets at a time until it does -- the same names stand for other states, and no row is served an old mask."""
    import paper_2506_01151_amd as zf
    torch = torch_cuda
    g = grammars.json_grammar()
    toks = [bytes([c]) for c in range(128)] + [b"tr", b"true", b'":', b"[[", b"}]", b"],"]
    off, data = wvocab.vocab_csr(toks)
    orc = oracle_lib.Oracle(g)
    eng = zf.Engine(g, toks, device=0, precompute_states=-1)
    prefixes = [b"[", b'{"k":"', b"[1,", b"tr", b'["\\u00', b"-1.5e", b'{"a"', b"[[[", b'{"a":1', b'[{"b":[']
    wants = []
    for p in prefixes:
        so = orc.new_state()
        assert so.feed_bytes(p)
        wants.append(so.mask(off, data))
    order = list(range(len(prefixes)))
    d_mask = torch.empty((len(prefixes), eng.W), dtype=torch.int32, device="cuda")

    def masks(rows, ks):
        d_mask.fill_(0x5A5A5A5A)
        zf.compute_mask(eng, rows, d_mask)
        assert np.array_equal(d_mask.cpu().numpy().view(np.uint32), np.stack([wants[k] for k in ks]))
        r = eng.mask_report()
        return r.cache_hits, r.cache_misses

    def rows_at(ks):
        rows = []
        for k in ks:
            rows.append(eng.new_state())
            rows[-1].advance_bytes(prefixes[k])
        return rows

    old = rows_at(order)
    assert masks(old, order) == (0, len(order)) and masks(old, order) == (len(order), 0)
    fed = 0
    for k in range(19):                                      # 1,048,576 states are its bound, less the largest chart it takes in
        row = eng.new_state()
        row.advance_bytes(b'{"a":' * k + b"[" * 60000)
        fed += 60000
        del row
    assert fed > 1 << 20
    back = order[::-1]                                       # other states under the first names of the new automaton
    new = rows_at(back)
    assert masks(new, back) == (0, len(order)) and masks(new, back) == (len(order), 0)
    assert sum(masks(old, order)) == len(order)              # (these come back in through their charts, some under names of their own)

"""GPU parity at the edges of the kernels' ranges: grammars and sizes where a
level, a tile or a segment begins, ends or is just full.  Expected masks come
from the CPU oracle."""

import itertools
import time

import numpy as np
import pytest

import oracle
import synth_inputs as si
from synth_inputs.vocab import Vocab

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def xgm():
    import paper_2411_15100_amd as lib
    lib.load_library()
    return lib


@pytest.fixture(scope="module")
def wl():
    from paper_2411_15100_amd import workloads
    return workloads


def _stream():
    return int(torch.cuda.current_stream().cuda_stream)


def precedence_grammar(levels: int) -> str:
    """`levels` rules that each occur in one place only (so that every one of them forces the frame below it)."""
    ops = "+-*/%&|^~!@$;:,.?"
    text = ['root ::= "<" l0 ">" | "{" l0 "}" tail', 'tail ::= ("<" l0 ">")*']
    for k in range(levels):
        op = ops[k % len(ops)] + (ops[k // len(ops)] if k >= len(ops) else "")
        text.append(f'l{k} ::= l{k + 1} ("{op}" l{k + 1})*')
    text.append(f'l{levels} ::= [a-z0-9]+ | "(" l0 ")"')
    return "\n".join(text)


# 48 frames is the longest way down that is followed without a key of its own
@pytest.mark.parametrize("levels", [1, 2, 3, 12, 47, 48, 49, 60])
def test_forced_frames(xgm, wl, levels):
    text = precedence_grammar(levels)
    vocab = si.make_vocab("bpe", 2048, 3)
    g, og = xgm.Grammar(text, "root"), oracle.Grammar(text, "root")
    cache = xgm.Cache(g, wl.make_xgm_vocab(vocab))
    walker = wl.BatchWalker([cache] * 3, vocab, seed=levels, structural_bias=0.6)
    oms = [oracle.EarleyMatcher(og) for _ in range(3)]
    toks = vocab.tokens()
    resident = xgm.DeviceBatch(walker.matchers, history=1, stream=_stream())
    d_mask = torch.zeros_like(walker.d_mask)
    for step in range(14):
        words = walker.fill()
        if xgm.fill_overflow_fixup(_stream()):
            words = walker.d_mask.cpu().numpy()
        want = oracle.pack_bitmask(np.stack([om.mask(vocab) for om in oms]))
        assert np.array_equal(words, want), f"step {step}"
        resident.fill_next_token_bitmask(d_mask.data_ptr(), _stream())
        resident.fill_overflow_fixup(_stream())
        assert np.array_equal(d_mask.cpu().numpy(), want), f"step {step}, resident states"
        picks = walker.step(words)
        ids = [int(t) if walker.history[b] else -1 for b, t in enumerate(picks)]
        resident.accept_tokens(torch.tensor(ids, dtype=torch.int32, device="cuda").data_ptr(), _stream())
        status = resident.status(_stream())
        for b in range(3):
            if not walker.history[b]:
                oms[b] = oracle.EarleyMatcher(og)
            else:
                assert oms[b].advance(toks[int(picks[b])])
            if not walker.history[b] or status[b]:
                resident.set_row(b, walker.matchers[b], _stream())


# Host-side states go along with the launch while they fit: 64 words (one row, a few frames), 896 words (a few dozen
# rows, or a deep stack); beyond that they are staged.  Rows with several stacks, ended rows, several grammars.
@pytest.mark.parametrize("rows,depth", [(1, 1), (1, 20), (1, 40), (1, 90), (1, 1700), (1, 1780), (2, 3), (9, 8), (28, 6), (33, 6), (45, 6), (70, 3), (130, 2)])
def test_states_in_the_launch(xgm, wl, rows, depth):
    vocab = si.make_vocab("bpe", 1500, 5)
    xv = wl.make_xgm_vocab(vocab)
    texts = [si.JSON_GRAMMAR, si.PYDSL_GRAMMAR, si.make_schema_grammar(1)]
    starts = [b"[" * depth, b"v" + b"[v" * min(depth, 3), b""]
    n = 1 if rows == 1 else 3
    caches = [xgm.Cache(xgm.Grammar(t, "root"), xv) for t in texts[:n]]
    ogs = [oracle.Grammar(t, "root") for t in texts[:n]]
    rng = np.random.Generator(np.random.PCG64(rows * 1000 + depth))
    toks = vocab.tokens()
    ms, oms = [], []
    for b in range(rows):
        k = b % n
        m, om = xgm.Matcher(cache=caches[k]), oracle.EarleyMatcher(ogs[k])
        if starts[k]:
            m.accept_bytes(starts[k])
            assert om.advance(starts[k])
        for _ in range(int(rng.integers(0, 4))):
            ids = np.flatnonzero(om.mask(vocab))
            ids = ids[ids != vocab.stop_ids[0]]
            t = int(rng.choice(ids)) if ids.size else None
            if t is not None:
                m.accept_token(t)
                assert om.advance(toks[t])
        ms.append(m)
        oms.append(om)
    want = np.stack([om.mask(vocab) for om in oms])
    if rows > 2:   # an ended row
        ms[2] = xgm.Matcher(cache=caches[0])
        ms[2].accept_bytes(b"null")
        ms[2].accept_token(int(vocab.stop_ids[0]))
        want[2] = False
        want[2, vocab.stop_ids] = True
    bits = oracle.pack_bitmask(want)
    masks = [torch.full((rows, xgm.bitmask_words(vocab.size)), -1, dtype=torch.int32, device="cuda") for _ in range(4)]
    logits = [torch.randn((rows, 1504), device="cuda").to(dt) for dt in (torch.bfloat16, torch.float32)]
    before = [t.cpu() for t in logits]
    xgm.fill_next_token_bitmask(ms, masks[0].data_ptr(), _stream())
    xgm.fill_next_token_bitmask_static(ms, masks[1].data_ptr(), _stream())
    xgm.fill_and_apply(ms, masks[2].data_ptr(), logits[0].data_ptr(), xgm.DTYPE_BF16, 1504, 1504, stream=_stream())
    xgm.fill_and_apply(ms, masks[3].data_ptr(), logits[1].data_ptr(), xgm.DTYPE_F32, 1504, 1504, stream=_stream())
    xgm.fill_overflow_fixup(_stream())
    torch.cuda.synchronize()
    for k in range(4):
        assert np.array_equal(masks[k].cpu().numpy(), bits), f"call {k}"
    allowed = torch.from_numpy(np.pad(want, ((0, 0), (0, 4))))
    for t, was in zip(logits, before):
        assert torch.equal(t.cpu(), torch.where(allowed, was, torch.full_like(was, float("-inf"))))


# A number that ends an expression leaves hundreds of tokens to the walk: few, as many as the queue
# of a workgroup holds (1024), more; in one segment and in several, whole or shared by workgroups (few rows).
@pytest.mark.parametrize("V", [300, 900, 1000, 1100, 1300, 2047, 2049, 6145, 8191, 8193, 24000, 90000])
def test_walk_entries(xgm, wl, V):
    vocab = si.make_vocab("bpe", V, 7)
    cache = xgm.Cache(xgm.Grammar(si.PYDSL_GRAMMAR, "root"), wl.make_xgm_vocab(vocab))
    og = oracle.Grammar(si.PYDSL_GRAMMAR, "root")
    texts = [b"x=1", b"if v==1:x=(1", b"while x:v[1", b"x=\"a", b"def v(x):return v[1]+1"]
    ms, oms = [], []
    for t in texts:
        m, om = xgm.Matcher(cache=cache), oracle.EarleyMatcher(og)
        m.accept_bytes(t)
        assert om.advance(t)
        ms.append(m)
        oms.append(om)
    want = oracle.pack_bitmask(np.stack([om.mask(vocab) for om in oms]))
    before = xgm.overflow_total()
    for rows in ([0], [1, 3, 4], [0, 1, 2, 3, 4], [k % 5 for k in range(100)]):
        d_mask = torch.full((len(rows), xgm.bitmask_words(V)), -1, dtype=torch.int32, device="cuda")
        xgm.fill_next_token_bitmask([ms[k] for k in rows], d_mask.data_ptr(), _stream())
        assert np.array_equal(d_mask.cpu().numpy(), want[rows]), f"host-side states, {len(rows)} rows"
        resident = xgm.DeviceBatch([ms[k] for k in rows], history=0, stream=_stream())
        d_mask.fill_(-1)
        resident.fill_next_token_bitmask(d_mask.data_ptr(), _stream())
        assert np.array_equal(d_mask.cpu().numpy(), want[rows]), f"resident states, {len(rows)} rows"
    assert xgm.overflow_total() == before


# Four workgroups share a segment, of 512 threads or, where there are more than 2560 of them and the tables are small
# (scripting grammar, not the C/SQL-like one), of 256; more than 1024 segments are not shared.
@pytest.mark.parametrize("script_only", [True, False])
@pytest.mark.parametrize("rows", [160, 161, 256, 257])
def test_walk_entries_of_large_batches(xgm, wl, rows, script_only):
    vocab = si.make_vocab("bpe", 30000, 7)
    xv = wl.make_xgm_vocab(vocab)
    states = [(0, b"x=1"), (0, b"if v==1:x=(1"), (0, b"while x:v[1"), (0, b"x=\"a"), (0, b"def v(x):return v[1]+1"), (0, b"")]
    if not script_only:
        states += [(1, b"int x"), (1, b""), (1, b"int x;")]
    texts = [si.PYDSL_GRAMMAR, si.CSQL_GRAMMAR]
    caches, ogs = [xgm.Cache(xgm.Grammar(t, "root"), xv) for t in texts], [oracle.Grammar(t, "root") for t in texts]
    ms, oms = [], []
    for k, t in states:
        m, om = xgm.Matcher(cache=caches[k]), oracle.EarleyMatcher(ogs[k])
        if t:
            if m.try_accept_bytes(t) != 0:
                continue
            assert om.advance(t)
        ms.append(m)
        oms.append(om)
    assert len(ms) >= len(states) - 1
    want = np.stack([om.mask(vocab) for om in oms])
    which = [(5 * b + b // 7) % len(ms) for b in range(rows)]
    bits, allowed = oracle.pack_bitmask(want)[which], torch.from_numpy(np.pad(want, ((0, 0), (0, 16))))[which]
    before = xgm.overflow_total()
    resident = xgm.DeviceBatch([ms[k] for k in which], history=0, stream=_stream())
    d_mask = torch.full((rows, xgm.bitmask_words(vocab.size)), -1, dtype=torch.int32, device="cuda")
    resident.fill_next_token_bitmask(d_mask.data_ptr(), _stream())
    assert np.array_equal(d_mask.cpu().numpy(), bits), "resident states"
    d_mask.fill_(-1)
    xgm.fill_next_token_bitmask([ms[k] for k in which], d_mask.data_ptr(), _stream())
    assert np.array_equal(d_mask.cpu().numpy(), bits), "host-side states"
    for dt, code in ((torch.bfloat16, xgm.DTYPE_BF16), (torch.float32, xgm.DTYPE_F32)):
        logits = torch.randn((rows, 30016), device="cuda").to(dt)
        was = logits.cpu()
        d_mask.fill_(-1)
        resident.fill_and_apply(d_mask.data_ptr(), logits.data_ptr(), code, 30016, 30016, stream=_stream())
        assert np.array_equal(d_mask.cpu().numpy(), bits), "one launch"
        assert torch.equal(logits.cpu(), torch.where(allowed, was, torch.full_like(was, float("-inf")))), dt
    assert xgm.overflow_total() == before


# Logits rows that begin anywhere: groups of 16 bytes in front of the row, behind it, and where the mask's words or a
# workgroup's 8192 elements end; rows narrower and wider than the mask.
@pytest.mark.parametrize("dtype_name", ["f32", "bf16"])
@pytest.mark.parametrize("V,Vl", [(1, 1), (3, 9), (32, 32), (33, 31), (8184, 8184), (8185, 8191), (8192, 8192), (8200, 8193), (16384, 16389), (24577, 24570)])
def test_apply_rows_that_begin_anywhere(xgm, dtype_name, V, Vl):
    code, ninf, udt, view = {"f32": (xgm.DTYPE_F32, 0xFF800000, np.uint32, np.int32), "bf16": (xgm.DTYPE_BF16, 0xFF80, np.uint16, np.int16)}[dtype_name]
    esize = np.dtype(udt).itemsize
    rng = np.random.Generator(np.random.PCG64(V + Vl))
    rows, total = 4, 6
    allowed = rng.random((rows, V)) < np.array([[0.5], [0.001], [0.999], [0.03]])
    d_mask = torch.from_numpy(oracle.pack_bitmask(allowed)).cuda()
    index = rng.permutation(total)[:rows].astype(np.int32)
    d_index = torch.from_numpy(index).cuda()
    want = np.zeros((rows, Vl), dtype=bool)
    want[:, :V] = allowed[:, :Vl] if Vl < V else allowed
    for offset in range(16 // esize):
        for stride in (Vl, Vl + 1, Vl + 6):
            before = rng.integers(0, 2 ** (8 * esize), size=offset + total * stride + 16, dtype=np.uint64).astype(udt)
            buf = torch.from_numpy(before.view(view)).cuda()
            xgm.apply_token_bitmask_inplace(buf.data_ptr() + offset * esize, code, total, Vl, stride, d_mask.data_ptr(), V, d_index.data_ptr(), rows,
                                            stream=_stream())
            expect = before.copy()
            for j, r in enumerate(index):
                row = expect[offset + r * stride:offset + r * stride + Vl]
                row[~want[j]] = ninf
            assert np.array_equal(buf.cpu().numpy().view(udt), expect), (offset, stride)


# The number of walk entries decides which kernel fills.  Builds share their temporary memory: these two, both of at most
# 32 nodes, 64 tokens and 64 list keys, lay it out alike, so that the second finds the first one's counters there.
def test_a_grammar_without_contexts_has_no_walk_entries(xgm, wl):
    toks = [b"[", b"]", b"x", b"y"] + [b"]" * k for k in range(2, 10)] + [b"q" * k for k in range(1, 52)] + [b""]
    assert len(toks) == 64

    class V_:
        data = np.frombuffer(b"".join(toks), dtype=np.uint8).copy()
        offsets = np.concatenate([[0], np.cumsum([len(t) for t in toks])]).astype(np.int64)
        stop_ids = np.array([63], dtype=np.int32)

    xv = wl.make_xgm_vocab(V_)
    nested = xgm.Grammar('root ::= "[" root "]" | "x"', "root")
    flat = xgm.Grammar('root ::= [xy]* "]"', "root")
    for _ in range(2):
        first = xgm.Cache(nested, xv)
    assert first.num_nodes <= 32 and first.stats["keys"] <= 64 and 0 < first.stats["context_dependent_pairs"] <= 64, first.stats
    assert first.debug_walk_entries() > 0
    second = xgm.Cache(flat, xv)
    assert second.num_nodes <= 32 and second.stats["context_dependent_pairs"] == 0
    assert second.debug_walk_entries() == 0


def rule_word(k: int) -> str:
    return "".join(chr(ord("a") + k // 26 ** j % 26) for j in range(3))


def many_rules_grammar(rules: int) -> str:
    """Brackets around words, each a rule of its own that may go on with others: tables of any size, tokens that are walked."""
    text = ['root ::= item ("," item)*', 'item ::= "[" root "]" | "{" root "}" | ' + " | ".join(f"k{k}" for k in range(rules))]
    return "\n".join(text + [f'k{k} ::= "{rule_word(k)}" ("(" k{k * 7 % rules} ")" | k{k * 5 % rules} "." )?' for k in range(rules)])


# A fill that walks stages the tables of the caches that have walk entries as far as they fit 31 KB: all of them, without
# the last headers, without the sections in front of those (1000 rules have 32 KB of FOLLOW sets); beside a row with
# small tables.
@pytest.mark.parametrize("rules", [1, 60, 500, 800, 900, 1000, 1400])
def test_walks_by_tables_of_all_sizes(xgm, wl, rules):
    text, name = many_rules_grammar(rules), rule_word
    toks = [bytes([c]) for c in b"[]{}(),.abcdefghijklmnopqrstuvwxyz"] + [b"]" * k for k in range(2, 40)] + [b"]}" * k for k in range(1, 20)]
    toks += [b"]]}]]," + name(k).encode() for k in range(0, rules, 1 + rules // 30)] + [b"]]]]]][[", b"]]]]]],aaa", b""]

    class V_:
        data = np.frombuffer(b"".join(toks), dtype=np.uint8).copy()
        offsets = np.concatenate([[0], np.cumsum([len(t) for t in toks])]).astype(np.int64)
        stop_ids = np.array([len(toks) - 1], dtype=np.int32)

    xv = wl.make_xgm_vocab(V_)
    texts = [text, si.JSON_GRAMMAR]
    caches = [xgm.Cache(xgm.Grammar(t, "root"), xv) for t in texts]
    ogs = [oracle.Grammar(t, "root") for t in texts]
    assert all(c.debug_walk_entries() > 0 for c in caches)
    starts = [(0, b"[[[[[[aaa"), (1, b"[[[[[[1"), (0, b"[[{[[[[{[[aaa"), (0, b"aaa"), (1, b'{"a":[[[[[[{"b":1'), (0, b"[" * 30 + b"aaa")]
    ms, want = [], []
    for k, start in starts:
        m, om = xgm.Matcher(cache=caches[k]), oracle.EarleyMatcher(ogs[k])
        m.accept_bytes(start)
        assert om.advance(start)
        ms.append(m)
        want.append(om.mask(V_))
    want = np.stack(want)
    bits = oracle.pack_bitmask(want)
    columns = (len(toks) + 7) // 8 * 8
    for rows in ([0, 1, 2, 3, 4, 5], [0], [1, 4], [b % 6 for b in range(300)]):
        some = [ms[b] for b in rows]
        resident = xgm.DeviceBatch(some, history=0, stream=_stream())
        d_mask = torch.full((len(rows), bits.shape[1]), -1, dtype=torch.int32, device="cuda")
        calls = [lambda lg: xgm.fill_next_token_bitmask(some, d_mask.data_ptr(), _stream()),
                 lambda lg: resident.fill_next_token_bitmask(d_mask.data_ptr(), _stream()),
                 lambda lg: xgm.fill_and_apply(some, d_mask.data_ptr(), lg.data_ptr(), xgm.DTYPE_F32, columns, columns, _stream()),
                 lambda lg: resident.fill_and_apply(d_mask.data_ptr(), lg.data_ptr(), xgm.DTYPE_F32, columns, columns, _stream())]
        for k, call in enumerate(calls):
            d_mask.fill_(-1)
            logits = torch.ones((len(rows), columns), device="cuda")
            call(logits)
            assert np.array_equal(d_mask.cpu().numpy(), bits[rows]), (rows[:8], k)
            if k >= 2:
                assert np.array_equal(logits.cpu().numpy()[:, :len(toks)] == 1.0, want[rows]), (rows[:8], k)
        assert xgm.debug_fill_count_steps(xgm.MatcherBatch(some), d_mask.data_ptr(), _stream()) > 0
        assert np.array_equal(d_mask.cpu().numpy(), bits[rows])


# Walks over the limits in fills whose states went along with the launch (2 rows) and whose states were staged (200),
# in the ring and in the static array, decided by one fixup.
@pytest.mark.parametrize("rows", [2, 200])
def test_records_of_launched_and_staged_states_are_fixed_up(xgm, wl, rows):
    deep = b")+" + b"(" * 30          # closes one level, then opens 30: more than 64 frames in one token
    toks = [b"1", b"(", b")", b"+", deep, deep + b"+", b"1" * 20, b")" * 40, b""]

    class V_:
        data = np.frombuffer(b"".join(toks), dtype=np.uint8).copy()
        offsets = np.concatenate([[0], np.cumsum([len(t) for t in toks])]).astype(np.int64)
        stop_ids = np.array([8], dtype=np.int32)

    cache = xgm.Cache(xgm.Grammar(si.ARITH_GRAMMAR, "expr"), wl.make_xgm_vocab(V_))
    og = oracle.Grammar(si.ARITH_GRAMMAR, "expr")
    states = []
    for text in (b"(" * 41 + b"1", b"1+", b"(" * 37 + b"1"):
        m, om = xgm.Matcher(cache=cache), oracle.EarleyMatcher(og)
        m.accept_bytes(text)
        assert om.advance(text)
        states.append((m, om.mask(V_)))
    which = [[(b + k) % 3 for b in range(rows)] for k in range(3)]
    d = [torch.full((rows, 1), -1, dtype=torch.int32, device="cuda") for _ in range(3)]
    logits = torch.ones((rows, 16), device="cuda")
    ms = [[states[k][0] for k in w] for w in which]
    xgm.fill_overflow_fixup(_stream())
    xgm.fill_next_token_bitmask(ms[0], d[0].data_ptr(), _stream())
    xgm.fill_next_token_bitmask_static(ms[1], d[1].data_ptr(), _stream())
    xgm.fill_and_apply(ms[2], d[2].data_ptr(), logits.data_ptr(), xgm.DTYPE_F32, 16, 16, stream=_stream())
    torch.cuda.synchronize()
    undecided_of = [sum(k != 1 for k in w) * 2 for w in which]   # tokens 4 and 5, where a parenthesis is open
    undecided = sum(undecided_of)
    want = [np.stack([states[k][1] for k in w]) for w in which]
    assert all(w[4] and not w[5] for k, (_, w) in enumerate(states) if k != 1)
    for k in range(3):                                      # left out, or in the one launch left allowed, until they are decided
        got = d[k].cpu().numpy()[:, 0].astype(np.uint32)
        for b, s in enumerate(which[k]):
            assert (got[b] >> 4) & 3 == (0 if s == 1 or k < 2 else 3), (k, b)
    assert xgm.fill_overflow_fixup(_stream()) == undecided
    for k in range(3):
        assert np.array_equal(d[k].cpu().numpy(), oracle.pack_bitmask(want[k])), k
    # records of the last eight fills are decided, those of the ninth and of an earlier static one are reported
    for more in (7, 8):
        xgm.fill_next_token_bitmask(ms[0], d[0].data_ptr(), _stream())
        for _ in range(more):
            xgm.fill_next_token_bitmask([states[1][0]], d[1].data_ptr(), _stream())
        if more == 7:
            assert xgm.fill_overflow_fixup(_stream()) == undecided_of[0]
            assert np.array_equal(d[0].cpu().numpy(), oracle.pack_bitmask(want[0]))
        else:
            with pytest.raises(xgm.XgmError) as e:
                xgm.fill_overflow_fixup(_stream())
            assert e.value.status == -9
    xgm.fill_next_token_bitmask_static(ms[1], d[1].data_ptr(), _stream())
    xgm.fill_next_token_bitmask_static([states[1][0]], d[0].data_ptr(), _stream())
    with pytest.raises(xgm.XgmError):
        xgm.fill_overflow_fixup(_stream())
    assert xgm.fill_overflow_fixup(_stream()) == 0


# The accept kernel walks by whole waves and puts candidates in order all pairs at once; its tables are staged as far as
# they fit 64 KB (the last grammar's FOLLOW sets alone take 70).  Random grammars, tokens allowed and not: the host
# engine's verdicts and its stacks in its order.
@pytest.mark.parametrize("seed", [1, 2])
def test_device_accept_gives_the_engines_stacks(xgm, wl, seed):
    from test_host_library import AMBIGUOUS_GRAMMAR, _random_grammar_text
    rng = np.random.Generator(np.random.PCG64(seed))
    toks = [b"a", b"b", b"c", b"d", b"(", b")", b"ab", b"ba", b"a(", b")b", b"cd)", b"((", b"))", b"abc", b"dcba", b"(a)", b"aa", b"aaa", b"x", b"y",
            b"z", b"ax", b"aay(", b"y(a", b"az", b"[", b"]", b"{", b"}", b"[[[{", b"}]", b"]]],", b"]]]],[", b"aaa(", b"e", b"f", b",", b".", b"bcd"]
    toks += [rule_word(k).encode() for k in range(0, 2200, 40)] + [b"[" + rule_word(k).encode() + b"]," for k in range(0, 2200, 300)] + [b""]

    class V_:
        data = np.frombuffer(b"".join(toks), dtype=np.uint8).copy()
        offsets = np.concatenate([[0], np.cumsum([len(t) for t in toks])]).astype(np.int64)
        stop_ids = np.array([len(toks) - 1], dtype=np.int32)

    xv = wl.make_xgm_vocab(V_)
    texts = [AMBIGUOUS_GRAMMAR, many_rules_grammar(2200)]
    while len(texts) < 60:
        text = _random_grammar_text(rng)
        try:
            xgm.Grammar(text, "root")
        except xgm.XgmError:
            continue
        texts.append(text)
    caches = [xgm.Cache(xgm.Grammar(t, "root"), xv) for t in texts]
    n_ok = n_rejected = n_multi = n_host = 0
    for walk in range(3):
        ms = [xgm.Matcher(cache=c) for c in caches]
        read = [xgm.Matcher(cache=c) for c in caches]
        batch = xgm.DeviceBatch(ms, history=1, stream=_stream())
        mask = torch.zeros((len(ms), xgm.bitmask_words(len(toks))), dtype=torch.int32, device="cuda")
        done = [False] * len(ms)
        for step in range(14):
            batch.fill_next_token_bitmask(mask.data_ptr(), _stream())
            batch.fill_overflow_fixup(_stream())
            allowed = wl.unpack_rows(mask.cpu().numpy(), len(toks))
            ids = np.full(len(ms), -1, dtype=np.int32)
            for b in range(len(ms)):
                some = np.flatnonzero(allowed[b])
                if not done[b]:
                    ids[b] = rng.integers(0, len(toks)) if some.size == 0 or rng.random() < 0.2 else some[rng.integers(0, some.size)]
            batch.accept_tokens(torch.from_numpy(ids).cuda().data_ptr(), _stream())
            status = batch.status(_stream())
            for b in range(len(ms)):
                if ids[b] < 0:
                    continue
                rc = ms[b].try_accept_token(int(ids[b]))
                if rc == -8 or (rc == 0 and status[b] in (-8, -9)):   # beyond the host's, or the device's, limits
                    n_host += 1
                    done[b] = True
                    continue
                assert status[b] == rc, (texts[b], toks[ids[b]], status[b], rc)
                n_ok += rc == 0
                n_rejected += rc == -6
                batch.get_row(b, read[b], _stream())
                assert read[b].is_terminated() == ms[b].is_terminated()
                if ms[b].is_terminated():
                    done[b] = True
                    continue
                stacks = [ms[b].stack(s) for s in range(ms[b].num_stacks())]
                assert [read[b].stack(s) for s in range(read[b].num_stacks())] == stacks, (texts[b], toks[ids[b]])
                n_multi += len(stacks) > 1
    assert n_ok > 500 and n_rejected > 200 and n_multi > 50, (n_ok, n_rejected, n_multi, n_host)


# Only nodes that can be on top of a stack have per-context lists: inside a rule whose start is entered again, behind calls
# in tail position, at a rule's end (also at the bottom of the stack).  Every state of up to five bytes.
@pytest.mark.parametrize("text", ['root ::= "(" a ")" "."\na ::= ("x" "y")* "z"', 'root ::= "(" b\nb ::= "x" b | "[" root "]" | ")"',
                                  'root ::= a "," a | "(" root ")"\na ::= "x" a | "x" | "[" a "]"', 'root ::= "(" c c ")"\nc ::= "x"* "y" | "[" root "]"'])
def test_every_top_has_its_lists(xgm, wl, text):
    alphabet = b"()[]xyz.,"
    toks = [bytes(t) for n in (1, 2, 3) for t in itertools.product(alphabet, repeat=n)] + [b"))))", b"]]]]", b")])])", b""]

    vocab = Vocab(np.frombuffer(b"".join(toks), dtype=np.uint8).copy(), np.cumsum([0] + [len(t) for t in toks]).astype(np.int64),
                  np.array([len(toks) - 1], dtype=np.int32))
    cache, og = xgm.Cache(xgm.Grammar(text, "root"), wl.make_xgm_vocab(vocab)), oracle.Grammar(text, "root")
    ms, want, texts = [], [], [b""]
    for t in texts:
        om = oracle.EarleyMatcher(og)
        if t and not om.advance(t):
            continue
        m = xgm.Matcher(cache=cache)
        if t:
            m.accept_bytes(t)
        ms.append(m)
        want.append(om.mask(vocab))
        if len(t) < 5:
            texts += [t + bytes([c]) for c in alphabet]
    want = oracle.pack_bitmask(np.stack(want))
    resident = xgm.DeviceBatch(ms, history=0, stream=_stream())
    for fill in (lambda d: xgm.fill_next_token_bitmask(ms, d, _stream()), lambda d: resident.fill_next_token_bitmask(d, _stream())):
        d_mask = torch.full((len(ms), xgm.bitmask_words(len(toks))), -1, dtype=torch.int32, device="cuda")
        fill(d_mask.data_ptr())
        assert np.array_equal(d_mask.cpu().numpy(), want)


# The classify kernel looks at 64 tokens and 64 nodes at a time, and at what a run of at least 16 tokens with the same first
# byte has in common (15 bytes of it at most): runs that begin and end anywhere in an item, grammars of one block of nodes
# and of several, tokens longer than a walk takes.
@pytest.mark.parametrize("run", [1, 15, 16, 17, 63, 64, 65, 200])
@pytest.mark.parametrize("words, nodes", [(11, 62), (12, 65), (40, 151)])
def test_classes_of_tokens_that_share_prefixes(xgm, wl, run, words, nodes):
    text = 'root ::= "{" ws item (ws "," ws item)* ws "}"\nws ::= " "*\nname ::= [a-z]+ | "-" name\nitem ::= ' + " | ".join(
        f'"{rule_word(k)}{rule_word(7 * k)}" ws ":" ws {"name" if k % 2 else "item"}' for k in range(words)) + ' | "." name'
    toks = [bytes([c]) for c in b"{}(),.:- abz"] + [b""]
    for p in (b" ", b"  ", b"a", b"aaa", b"  }", b"abcdefghijklmn", b"abcdefghijklmno", b"abcdefghijklmnopq", b" aaaaaa : aaaaaa", b", .", b"---"):
        toks += [p + rule_word(k).encode() for k in range(run - 1)] + [p]
    if run == 64:
        toks += [b"a" * 300, b"-" * 256 + b"a", b" " * 280]  # (each decided on the host, its neighbours by their walks)
    toks = list(dict.fromkeys(toks))
    stop = toks.index(b"")
    vocab = Vocab(np.frombuffer(b"".join(toks), dtype=np.uint8).copy(), np.cumsum([0] + [len(t) for t in toks]).astype(np.int64),
                  np.array([stop], dtype=np.int32))
    g, og = xgm.Grammar(text, "root"), oracle.Grammar(text, "root")
    assert g.num_nodes == nodes
    cache = xgm.Cache(g, wl.make_xgm_vocab(vocab), keep_plain=True)
    assert (cache.host_classified > 0) == (run == 64)
    for node in range(g.num_nodes):
        want = og.classify(g.rule_name(g.node_rule(node)), g.node_path(node), vocab)
        acc, unc = cache.copy_node_bits(node)
        for got, cls in ((acc, 2), (unc, 1), (cache.copy_node_plain(node), 4)):
            assert np.array_equal(got, oracle.pack_bitmask(want == cls)), (node, cls)
        assert cache.num_uncertain(node) == int((want == 1).sum()) and cache.num_uncertain_plain(node) == int((want == 4).sum())


# A build keeps only the words of its rank-space rows that are not zero, unless it keeps the context-dependent bitsets too or
# goes through the nodes in batches (of 32 here, the last one smaller): the same caches from all three, and the oracle's masks;
# vocabularies that end anywhere in an item of 64 tokens, in 64 items and in 64 times 64 of them, and the largest one.
@pytest.mark.parametrize("V", [37, 64, 65, 511, 4095, 4097, 8193, 262145, 589824])
@pytest.mark.parametrize("family", ["json", "words"])
def test_builds_of_all_kinds_give_the_same_cache(xgm, wl, family, V):
    text, nodes = si.JSON_GRAMMAR, 74
    if family == "words":
        n, nodes = 18, 101
        text = 'root ::= ([a-z] [a-z]* | [0-9]+ | " " | "-" word)* "." | "(" root ")" tail\ntail ::= ("," root)*\nword ::= '
        text += " | ".join(f"w{k}" for k in range(n)) + "".join(f'\nw{k} ::= "{rule_word(7 * k)}" " "* [0-9]' for k in range(n))
    chars = bytes(range(33, 127)) if V > 50000 else b'{}[]:,"0123456789.E+- ()abcdefgxyz\\'
    toks = [bytes(t) for n in (1, 2, 3) for t in itertools.islice(itertools.product(chars, repeat=n), V)]
    toks = (toks[:V - 1] if V < 50000 else toks[:V - 1] + [b"%d" % k for k in range(10 ** 6, 10 ** 6 + max(0, V - 1 - len(toks)))]) + [b""]
    vocab = Vocab(np.frombuffer(b"".join(toks), dtype=np.uint8).copy(), np.cumsum([0] + [len(t) for t in toks]).astype(np.int64),
                  np.array([len(toks) - 1], dtype=np.int32))
    assert vocab.size == V and len(set(toks)) == V
    g, og, xv = xgm.Grammar(text, "root"), oracle.Grammar(text, "root"), wl.make_xgm_vocab(vocab)
    assert g.num_nodes == nodes and nodes > 64 and nodes % 32
    caches = [xgm.Cache(g, xv), xgm.Cache(g, xv, keep_plain=True)]
    xgm.debug_set_build_batch_nodes(32)
    try:
        caches.append(xgm.Cache(g, xv))
    finally:
        xgm.debug_set_build_batch_nodes(0)
    for node in range(g.num_nodes):
        acc, _ = caches[0].copy_node_bits(node, with_uncertain=False)
        for c in caches[1:]:
            assert np.array_equal(c.copy_node_bits(node, with_uncertain=False)[0], acc)
            assert c.num_uncertain(node) == caches[0].num_uncertain(node)
            assert c.num_uncertain_plain(node) == caches[0].num_uncertain_plain(node)
    assert caches[0].stats == caches[1].stats == caches[2].stats
    starts = [b"", b"[", b'{"a', b'{"a":[1', b"[[[-2.", b'["b",']
    if family == "words":
        starts = [b"", b"a", b"(12", b"((b ", b"(c.)", b"(c.),d", b"(a -", b"-h", b"((-aaa  ", b"(-aaa 1-haa"]
    want = []
    for start in starts:
        om = oracle.EarleyMatcher(og)
        assert om.advance(start)
        want.append(om.mask(vocab))
    want = oracle.pack_bitmask(np.stack(want))
    for kind, c in enumerate(caches):
        ms = []
        for start in starts:
            ms.append(xgm.Matcher(cache=c))
            if start:
                ms[-1].accept_bytes(start)
        d_mask = torch.full((len(ms), xgm.bitmask_words(V)), -1, dtype=torch.int32, device="cuda")
        xgm.fill_next_token_bitmask(ms, d_mask.data_ptr(), _stream())
        assert np.array_equal(d_mask.cpu().numpy(), want), kind


# The list kernels take the pairs of a node 64 at a time and the contexts of its rule 64 and 256 at a time: a rule in m places,
# as many tokens that begin with the same byte and go on to the next, or to the end and to what follows it.
@pytest.mark.parametrize("m", [1, 7, 8, 9, 63, 64, 65, 257])
@pytest.mark.parametrize("pairs", [1, 16, 63, 64, 65, 300])
def test_contexts_and_pairs_of_all_counts(xgm, wl, m, pairs):
    text = 'root ::= item (";" item)*\nws ::= " "+\nitem ::= ' + " | ".join(f'"{rule_word(k)}" ws "{rule_word(5 * k)}" ws' for k in range(m))
    text += ' | "(" ws root ")"'
    toks = [bytes([c]) for c in b"();. abcdefghij"] + [b" " * k for k in (2, 3, 17)] + [b" ;", b" );", b" ) ;"]
    for k in range(pairs):
        toks += [p + rule_word(5 * k).encode() for p in (b" ", b"   ", b" ;", b" " * 14)]
        toks += [b" " + rule_word(5 * k)[:2].encode(), b" " + rule_word(5 * k).encode() + b" ;" + rule_word(k).encode(),
                 b" )" + rule_word(k).encode()]
    toks = list(dict.fromkeys(toks)) + [b""]
    vocab = Vocab(np.frombuffer(b"".join(toks), dtype=np.uint8).copy(), np.cumsum([0] + [len(t) for t in toks]).astype(np.int64),
                  np.array([len(toks) - 1], dtype=np.int32))
    cache, og = xgm.Cache(xgm.Grammar(text, "root"), wl.make_xgm_vocab(vocab)), oracle.Grammar(text, "root")
    ms, want = [], []
    for k in sorted({0, 1, 7, 8, 62, 63, 64, 65, 255, 256, m - 1} & set(range(m))):
        for start in (rule_word(k) + " ", rule_word(k) + " " + rule_word(5 * k) + " ", "( (  " + rule_word(k) + " " + rule_word(5 * k) + "  "):
            ms.append(xgm.Matcher(cache=cache))
            ms[-1].accept_bytes(start.encode())
            om = oracle.EarleyMatcher(og)
            assert om.advance(start.encode())
            want.append(om.mask(vocab))
    d_mask = torch.full((len(ms), xgm.bitmask_words(len(toks))), -1, dtype=torch.int32, device="cuda")
    xgm.fill_next_token_bitmask(ms, d_mask.data_ptr(), _stream())
    assert np.array_equal(d_mask.cpu().numpy(), oracle.pack_bitmask(np.stack(want)))


# Neighbours in byte-sorted order with ids in different segments: the 64 pairs that a wave of the list kernels takes add to the
# counters of up to 64 segments, of accepted and of walk entries (with more than 32 segments a lane has several counters), and
# every wave takes many such groups, one after the other.
@pytest.mark.parametrize("depth", [0, 1, 2])
@pytest.mark.parametrize("V", [5000, 9000, 300000])
def test_lists_over_many_segments(xgm, wl, V, depth):
    m, seed = 24, V + depth
    text = 'root ::= item (";" item)*\nws ::= " "+\nitem ::= ' + " | ".join(f'"{rule_word(k)}" ws "{rule_word(5 * k)}" ws' for k in range(m))
    text += ' | "(" ws root ")"'
    toks = [bytes([c]) for c in b"();. abcdefghij"] + [b" " * k for k in (2, 3, 17)]
    for k in range(m):
        for j in range(40):   # (tokens that end in the second word, behind it, and behind one to three brackets)
            toks += [b" " + rule_word(5 * k).encode() + b" " * (j % 3) + b")" * (j // 3 % 4) + (b";" + rule_word(j % m).encode()) * (j // 12 % 2) + b" " * (j % 7)]
        toks += [b" " * (k % 3) + rule_word(5 * k)[:n].encode() for n in range(1, len(rule_word(5 * k)) + 1)]
    toks += [b" " * k + b";" + rule_word(j).encode() for k in range(8) for j in range(m)] + [b" " * (k % 9) + b")" * (k // 9 + 1) for k in range(90)]
    toks = list(dict.fromkeys(toks))
    toks += [b"~%d" % k for k in range(V - 1 - len(toks))]
    order = np.random.Generator(np.random.PCG64(seed)).permutation(len(toks))
    toks = [toks[k] for k in order] + [b""]
    vocab = Vocab(np.frombuffer(b"".join(toks), dtype=np.uint8).copy(), np.cumsum([0] + [len(t) for t in toks]).astype(np.int64),
                  np.array([len(toks) - 1], dtype=np.int32))
    assert vocab.size == V
    cache, og = xgm.Cache(xgm.Grammar(text, "root"), wl.make_xgm_vocab(vocab), depth=depth), oracle.Grammar(text, "root")
    assert depth == 0 or cache.debug_walk_entries() > 0
    ms, want = [], []
    for k in (0, 5, m - 1):
        for start in (rule_word(k) + " ", rule_word(k) + " " + rule_word(5 * k) + " ", "( ( ( " + rule_word(k) + " " + rule_word(5 * k) + " "):
            ms.append(xgm.Matcher(cache=cache))
            ms[-1].accept_bytes(start.encode())
            om = oracle.EarleyMatcher(og)
            assert om.advance(start.encode())
            want.append(om.mask(vocab))
    d_mask = torch.full((len(ms), xgm.bitmask_words(V)), -1, dtype=torch.int32, device="cuda")
    xgm.fill_next_token_bitmask(ms, d_mask.data_ptr(), _stream())
    assert np.array_equal(d_mask.cpu().numpy(), oracle.pack_bitmask(np.stack(want)))


# What a cache tells about a node is one copy, whether the node lists its accepted tokens or keeps a bitset; what it tells about
# a matcher's state takes the device only once.
def test_a_cache_is_read_with_few_copies(xgm, wl):
    vocab = si.make_vocab("bpe", 32000, 0)
    cache = xgm.Cache(xgm.Grammar(si.JSON_GRAMMAR, "root"), wl.make_xgm_vocab(vocab))

    def median(call):
        times = []
        for _ in range(101):
            t0 = time.perf_counter()
            call()
            times.append(time.perf_counter() - t0)
        return sorted(times)[50]

    accepted = [int(oracle.unpack_bitmask(cache.copy_node_bits(n, with_uncertain=False)[0], vocab.size).sum()) for n in range(cache.num_nodes)]
    listed = [n for n, k in enumerate(accepted) if k * 2 <= xgm.bitmask_words(vocab.size)]
    assert 0 < len(listed) < cache.num_nodes and max(accepted[n] for n in listed) > 0
    nodes = max(listed, key=lambda n: accepted[n]), max(range(cache.num_nodes), key=lambda n: accepted[n])
    of_list, of_bitset = (median(lambda: cache.copy_node_bits(n, with_uncertain=False)) for n in nodes)
    assert of_list < 2 * of_bitset
    m = xgm.Matcher(cache=cache)
    m.accept_bytes(b'{"a": [1, "x')
    assert median(m.debug_fill_work) < of_bitset


# Putting a state into a row is seven small copies and a launch, taking it out is four copies: at most 2.8 times as long (2.4
# measured; 3.1 with three more copies for the row's scalars, 2.5 with those and without a launch).
def test_a_state_goes_into_a_row_with_few_copies(xgm, wl):
    cache = xgm.Cache(xgm.Grammar(si.JSON_GRAMMAR, "root"), wl.make_xgm_vocab(si.make_vocab("bpe", 151936, 0)))
    m = xgm.Matcher(cache=cache)
    m.accept_bytes(b'{"a": [1, {"b": "x')
    batch = xgm.DeviceBatch([m] * 8, history=4, stream=_stream())
    times = {batch.set_row: [], batch.get_row: []}
    for _ in range(200):
        for call, ts in times.items():
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            call(5, m, _stream())
            ts.append(time.perf_counter() - t0)
    assert min(times[batch.set_row]) < 2.8 * min(times[batch.get_row])


# Few walks of a row go to waves, unless a cache of the batch (the markup grammar's) is known to walk to the limits.
@pytest.mark.parametrize("V", [4096, 32000])
def test_walks_by_waves_and_by_lanes(xgm, wl, V):
    vocab = si.make_vocab("bpe", V, 0)
    xv = wl.make_xgm_vocab(vocab)
    texts = [si.PYDSL_GRAMMAR, si.XML_GRAMMAR, si.CSQL_GRAMMAR]
    caches = [xgm.Cache(xgm.Grammar(t, "root"), xv) for t in texts]
    assert [c.host_classified > 0 for c in caches] == [False, True, False]
    starts = [(0, b"x=1"), (1, b"<a"), (2, b"int x"), (1, b"<a>x"), (0, b"if v==1:x=(1"), (1, b"<a><b"), (1, b"<a b=\"c")]
    ms, want = [], []
    for k, start in starts:
        m, om = xgm.Matcher(cache=caches[k]), oracle.EarleyMatcher(oracle.Grammar(texts[k], "root"))
        if m.try_accept_bytes(start) != 0:
            continue
        assert om.advance(start)
        ms.append((k, m))
        want.append(oracle.pack_bitmask(om.mask(vocab)))
    assert {k for k, _ in ms} == {0, 1, 2}
    everything = list(range(len(ms)))
    for rows in (everything, [b for b in everything if ms[b][0] != 1], [b for b in everything if ms[b][0] == 1]):
        some = [ms[b][1] for b in rows]
        resident = xgm.DeviceBatch(some, history=0, stream=_stream())
        for k in range(2):
            d_mask = torch.full((len(rows), xgm.bitmask_words(V)), -1, dtype=torch.int32, device="cuda")
            if k:
                resident.fill_next_token_bitmask(d_mask.data_ptr(), _stream())
                resident.fill_overflow_fixup(_stream())
            else:
                xgm.fill_next_token_bitmask(some, d_mask.data_ptr(), _stream())
                xgm.fill_overflow_fixup(_stream())
            assert np.array_equal(d_mask.cpu().numpy(), np.stack([want[b] for b in rows])), (rows, k)


# What a fill reads is kept until it is done, also where a program drops its matchers and caches right after the call: the
# library remembers 16 to 32 fills whose states went along with the launch (1 row), or were staged in the static array, and
# 8 that were staged elsewhere (200 rows), and waits for those before it forgets them.
@pytest.mark.parametrize("form,rows", [("fill", 1), ("fill", 200), ("fused", 1), ("fused", 200), ("static", 1), ("static", 200)])
def test_fills_are_forgotten_only_when_they_are_done(xgm, wl, form, rows):
    vocab = si.make_vocab("bpe", 2048, 3)
    m = xgm.Matcher(cache=xgm.Cache(xgm.Grammar(si.JSON_GRAMMAR, "root"), wl.make_xgm_vocab(vocab)))
    ms = [m] * rows
    d_mask = torch.zeros((rows, xgm.bitmask_words(2048)), dtype=torch.int32, device="cuda")
    logits = torch.zeros((rows, 2048), device="cuda")

    def call():
        if form == "fill":
            xgm.fill_next_token_bitmask(ms, d_mask.data_ptr(), _stream())
        elif form == "static":
            xgm.fill_next_token_bitmask_static(ms, d_mask.data_ptr(), _stream())
        else:
            xgm.fill_and_apply(ms, d_mask.data_ptr(), logits.data_ptr(), xgm.DTYPE_F32, 2048, 2048, _stream())

    for _ in range(9):
        call()
    big = torch.empty(1 << 30, dtype=torch.int32, device="cuda")   # 4 GiB: about a millisecond to fill
    torch.cuda.synchronize()
    for k in range(60):
        big.fill_(k)
    before = torch.cuda.Event()
    before.record()
    for _ in range(8):
        call()
    assert not before.query()
    for _ in range(25 if rows == 1 or form == "static" else 1):
        call()
    assert before.query()
    want = oracle.EarleyMatcher(oracle.Grammar(si.JSON_GRAMMAR, "root")).mask(vocab)
    assert np.array_equal(d_mask.cpu().numpy(), np.tile(oracle.pack_bitmask(want), (rows, 1)))


# A build does not wait for what other streams do (once its temporary memory is there), also where its tables take more than
# the pinned memory that the builds share: a rule used in n places of a rule that is used in n places has n * n contexts two
# frames down, 9 MB of keys for 1500.
@pytest.mark.parametrize("n", [100, 1500])
def test_builds_do_not_wait_for_other_streams(xgm, wl, n):
    text = "root ::= " + " ".join(f'w "{k:05d}"' for k in range(n)) + "\nw ::= " + " ".join(f'"{k:05d}" v' for k in range(n)) + "\nv ::= [a-z]+"
    vocab = si.make_vocab("bpe", 4096, 0)
    xv, g = wl.make_xgm_vocab(vocab), xgm.Grammar(text, "root")
    big = torch.empty(1 << 28, dtype=torch.int32, device="cuda")   # 1 GiB: 0.15 ms to fill
    waited = []
    for _ in range(6):
        # (a stream that shares its hardware queue with the other one waits for that; not all of them do)
        own, other = torch.cuda.Stream(), torch.cuda.Stream()
        for _ in range(2):
            cache = xgm.Cache(g, xv, int(own.cuda_stream))
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            for k in range(600):
                big.fill_(k)
            after = torch.cuda.Event()
            after.record()
        cache = xgm.Cache(g, xv, int(own.cuda_stream))
        waited.append(after.query())
        torch.cuda.synchronize()
    assert not all(waited)
    start = b"00000abc00001de" + b"".join(b"%05dx" % k for k in range(2, n)) + b"00000" + b"00000y"
    m, om = xgm.Matcher(cache=cache), oracle.EarleyMatcher(oracle.Grammar(text, "root"))
    m.accept_bytes(start)
    assert om.advance(start)
    d_mask = torch.full((1, xgm.bitmask_words(4096)), -1, dtype=torch.int32, device="cuda")
    xgm.fill_next_token_bitmask([m], d_mask.data_ptr(), _stream())
    assert np.array_equal(d_mask.cpu().numpy()[0], oracle.pack_bitmask(om.mask(vocab)))


# Fills on more streams than the library remembers launches of (4), in turn: those of the others are staged; after a thousand
# fills on one stream the others' places are taken over.
def test_fills_on_many_streams(xgm, wl):
    vocab = si.make_vocab("bpe", 2048, 3)
    caches = [xgm.Cache(xgm.Grammar(t, "root"), wl.make_xgm_vocab(vocab)) for t in (si.JSON_GRAMMAR,)]
    og = oracle.Grammar(si.JSON_GRAMMAR, "root")
    streams = [torch.cuda.Stream() for _ in range(7)]
    for lap in range(25):
        if lap in (8, 16):
            m = xgm.Matcher(cache=caches[0])
            some = torch.zeros((1, xgm.bitmask_words(2048)), dtype=torch.int32, device="cuda")
            for _ in range(1100):
                xgm.fill_next_token_bitmask([m], some.data_ptr(), int(streams[lap % 7].cuda_stream))
        texts = [b"[" * (1 + (lap + k) % 5) for k in range(7)]
        masks = [torch.full((2, xgm.bitmask_words(2048)), -1, dtype=torch.int32, device="cuda") for _ in streams]
        torch.cuda.synchronize()
        for form in (xgm.fill_next_token_bitmask, xgm.fill_next_token_bitmask_static):
            for s, t, d in zip(streams, texts, masks):
                m = xgm.Matcher(cache=caches[0])
                m.accept_bytes(t)
                if form is xgm.fill_next_token_bitmask_static:
                    torch.cuda.synchronize()   # (its calls share their staging: ordered by the caller)
                form([m], d[1 if form is xgm.fill_next_token_bitmask_static else 0:].data_ptr(), int(s.cuda_stream))
        torch.cuda.synchronize()
        for t, d in zip(texts, masks):
            om = oracle.EarleyMatcher(og)
            assert om.advance(t)
            assert np.array_equal(d.cpu().numpy(), np.tile(oracle.pack_bitmask(om.mask(vocab)), (2, 1)))

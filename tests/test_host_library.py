"""CPU tests of the library's host side: C-ABI surface, grammar compilation,
matcher state, error codes.  The automaton is compared with the oracle on
membership and on token classes (the oracle never sees the library's tables;
a node is named by its rule and a symbol path from the rule's start)."""

import ctypes
import os
import re
import sys
import sysconfig
import threading
import time
import zlib

import numpy as np
import pytest

import oracle
import paper_2411_15100_amd as xgm
from paper_2411_15100_amd import binding
import synth_inputs as si
from test_oracle_misc import TinyVocab

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

GRAMMARS = {
    "arith": (si.ARITH_GRAMMAR, "expr", b"0123456789+*() "),
    "json": (si.JSON_GRAMMAR, "root", b' \n"{}[],:\\/abfnrtu0123456789.eE+-\xc3\xa9\xe4\xb8\xad\xf0\x9f\x98\x80xyz'),
    "csql": (si.CSQL_GRAMMAR, "root", b" \n(){}[];,.*+-/%<>=!&|^~?:'\"\\_abcdefhilnorstuwxSELCTFROMWHNDBYGUPIAV0123459"),
    "xml": (si.XML_GRAMMAR, "root", b" \n\t<>/=\"'&;#!-._abcxyzAZ019"),
    "pydsl": (si.PYDSL_GRAMMAR, "root", b" \n()[]{}:;,.=+-*/%<>!~#'\"\\xzuv_ab019ifelsnotrdwhpcTFNm"),
    "schema": (si.make_schema_grammar(3), "root", b' \n"{}[],:\\abcdefghijklmnopqrstuvwxyz_0123456789.eE+-tfu'),
}


def test_every_declared_symbol_is_exported_and_bound():
    header = open(os.path.join(ROOT, "include", "xgm.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(xgm_[a-z_0-9]+)\s*\(", header))
    assert len(declared) >= 30
    lib = xgm.load_library()
    for name in declared:
        assert hasattr(lib, name), f"{name} is declared but not exported"
        assert name in binding.SIGNATURES, f"{name} has no binding"
    assert set(binding.SIGNATURES) == declared


@pytest.mark.parametrize("name", list(GRAMMARS))
def test_membership_matches_oracle_on_random_byte_walks(name):
    text, root, alphabet = GRAMMARS[name]
    g = xgm.Grammar(text, root)
    og = oracle.Grammar(text, root)
    rng = np.random.Generator(np.random.PCG64(zlib.crc32(name.encode())))
    n_accept = n_reject = 0
    for trial in range(12):
        m = xgm.Matcher(grammar=g)
        prefix = b""
        for step in range(60):
            assert m.can_terminate() == (og.recognize(prefix) == 2), prefix
            # try several random bytes; the oracle must agree on every verdict
            progressed = False
            for b in rng.permutation(list(alphabet))[:8]:
                cand = prefix + bytes([int(b)])
                rc = m.try_accept_bytes(bytes([int(b)]))
                want = og.recognize(cand) > 0
                assert (rc == 0) == want, (cand, rc)
                if rc == 0:
                    n_accept += 1
                    prefix = cand
                    progressed = True
                    break
                assert rc == -6  # TOKEN_REJECTED, state unchanged
                n_reject += 1
            if not progressed:
                # steer with the oracle's completion so the walk keeps going
                tail = oracle.EarleyMatcher(og)
                assert tail.advance(prefix)
                nxt = tail.completion()[:1]
                if not nxt:
                    break
                m.accept_bytes(nxt)
                prefix += nxt
    assert n_accept > 50 and n_reject > 100


def test_multibyte_chunks_equal_single_bytes():
    g = xgm.Grammar(si.JSON_GRAMMAR, "root")
    doc = '{"k\\u00e9": [1.5e3, "中\U0001f600", true, null, {"x": -0}]}'.encode()
    rng = np.random.Generator(np.random.PCG64(2))
    for _ in range(20):
        m = xgm.Matcher(grammar=g)
        pos = 0
        while pos < len(doc):
            k = int(rng.integers(1, 7))
            m.accept_bytes(doc[pos:pos + k])
            pos += k
        assert m.can_terminate()
        assert m.num_stacks() >= 1


def _classes_for_all_nodes(text, root, vocab, nodes=None):
    g = xgm.Grammar(text, root)
    og = oracle.Grammar(text, root)
    toks = vocab.tokens() if hasattr(vocab, "tokens") else vocab.toks
    seen = set()
    for node in (range(g.num_nodes) if nodes is None else nodes):
        rule = g.rule_name(g.node_rule(node))
        path = g.node_path(node)
        want = og.classify(rule, path, vocab)
        got = np.array([g.debug_classify_host(node, t) for t in toks], dtype=np.uint8)
        bad = np.flatnonzero(got != want)
        assert bad.size == 0, (rule, path, toks[bad[0]], int(got[bad[0]]), int(want[bad[0]]))
        seen |= set(got.tolist())
    return seen


def test_host_classes_match_oracle_arith_all_nodes():
    vocab = si.make_vocab("arith", 1024, 0)
    assert _classes_for_all_nodes(si.ARITH_GRAMMAR, "expr", vocab) == {0, 1, 2, 4}


def test_host_classes_match_oracle_json_all_nodes():
    import itertools
    alphabet = [b'"', b"\\", b"{", b"}", b"[", b"]", b",", b":", b" ", b"1", b"0", b"-", b".", b"e", b"t", b"r", b"u",
                b"a", b"\xc3", b"\xa9", b"\xf0", b"\x9f", b"n"]
    toks = [b"".join(t) for n in (1, 2) for t in itertools.product(alphabet, repeat=n)]
    toks += [b"true", b"null", b"fals", b'"ab"', b'":', b'",', b'"}', b"\\u00e9", b"1.5e3", b"", b"\xe4\xb8\xad", b"\xe4\xb8"]
    vocab = TinyVocab(toks)
    assert _classes_for_all_nodes(si.JSON_GRAMMAR, "root", vocab) == {0, 1, 2, 4}


def test_host_classes_match_oracle_csql_sample():
    vocab = si.make_vocab("bpe", 2048, 1)
    g = xgm.Grammar(si.CSQL_GRAMMAR, "root")
    rng = np.random.Generator(np.random.PCG64(4))
    nodes = sorted(set(int(n) for n in rng.integers(0, g.num_nodes, size=25)))
    _classes_for_all_nodes(si.CSQL_GRAMMAR, "root", vocab, nodes)


def test_compile_errors():
    def status(text, root="root"):
        with pytest.raises(xgm.XgmError) as e:
            xgm.Grammar(text, root)
        return e.value.status

    assert status('root ::= "a') == -2
    assert status("root ::= [a") == -2
    assert status('root ::= ("a"') == -2
    assert status('root ::= "a")') == -2
    assert status('root = "a"') == -2
    assert status("") == -2
    assert status('root ::= "a"\nroot ::= "b"') == -2
    assert status('root ::= "\\q"') == -2
    assert status("root ::= other") == -3
    assert status('a ::= "x"') == -3
    assert status('root ::= root "a" | "b"') == -4
    assert status('root ::= a "x" | "z"\na ::= b? root\nb ::= "y"') == -4      # hidden behind a nullable prefix
    assert status('root ::= "a" root') == -5
    assert status('root ::= dead\ndead ::= "x" dead') == -5


def test_left_recursion_rejection_is_conservative():
    """The library refuses left-recursive grammars; the oracle's Earley side
    takes them, which shows nothing else is affected by the refusal."""
    text = 'E ::= E "+" "n" | "n"'
    assert oracle.Grammar(text, "E").recognize(b"n+n") == 2
    with pytest.raises(xgm.XgmError) as e:
        xgm.Grammar(text, "E")
    assert e.value.status == -4


def test_unproductive_and_unreachable_parts_are_dropped():
    g = xgm.Grammar('root ::= "a" dead | "a" "b"\ndead ::= "x" dead\nunused ::= "zzz"', "root")
    assert g.num_rules == 1
    m = xgm.Matcher(grammar=g)
    m.accept_bytes(b"a")
    assert m.try_accept_bytes(b"x") == -6
    m.accept_bytes(b"b")
    assert m.can_terminate()


def test_nullable_rules_and_loops():
    text = 'root ::= (e | "a")* "b"\ne ::= "c"?'
    g = xgm.Grammar(text, "root")
    og = oracle.Grammar(text, "root")
    import itertools
    for n in range(0, 6):
        for tup in itertools.product(b"abc", repeat=n):
            s = bytes(tup)
            m = xgm.Matcher(grammar=g)
            ok = m.try_accept_bytes(s) == 0
            want = og.recognize(s)
            assert ok == (want > 0), s
            if ok:
                assert m.can_terminate() == (want == 2), s


def test_token_level_errors_and_termination():
    vocab = si.make_vocab("arith", 1024, 0)
    toks = vocab.tokens()
    index = {t: i for i, t in enumerate(toks)}
    stop = int(vocab.stop_ids[0])
    g = xgm.Grammar(si.ARITH_GRAMMAR, "expr")
    v = xgm.Vocab(vocab.data, vocab.offsets, vocab.stop_ids)
    m = xgm.Matcher(grammar=g, vocab=v)
    assert m.try_accept_token(stop) == -6          # empty text is not an expression
    assert m.try_accept_token(index[b")"]) == -6
    assert m.stack(0) == xgm.Matcher(grammar=g, vocab=v).stack(0)  # unchanged
    m.accept_token(index[b"1"])
    assert m.can_terminate() and not m.is_terminated()
    assert m.try_accept_token(-1) == -1 and m.try_accept_token(1024) == -1
    m.accept_token(stop)
    assert m.is_terminated() and m.num_stacks() == 0
    assert m.try_accept_token(index[b"1"]) == -7
    m.reset()
    assert not m.is_terminated() and m.num_stacks() == 1


def test_parallel_stacks_and_their_limit():
    # "1 " may continue the term or the expression: two parallel stacks
    g = xgm.Grammar(si.ARITH_GRAMMAR, "expr")
    m = xgm.Matcher(grammar=g)
    m.accept_bytes(b"1 ")
    assert m.num_stacks() == 2
    # nested binary choices that stay on the stack: 2^k stacks after k bytes
    rules = ['root ::= a | b', 'a ::= "x" root? "p"', 'b ::= "x" root? "q"']
    g2 = xgm.Grammar("\n".join(rules), "root")
    m2 = xgm.Matcher(grammar=g2)
    m2.accept_bytes(b"xxxxxx")
    assert m2.num_stacks() == 64
    before = [m2.stack(s) for s in range(64)]
    assert m2.try_accept_bytes(b"x") == -8
    assert [m2.stack(s) for s in range(64)] == before


def test_vocab_argument_checks():
    lib = xgm.load_library()
    h = ctypes.c_void_p()
    off = np.array([0, 1, 0], dtype=np.int64)
    data = np.zeros(4, dtype=np.uint8)
    assert lib.xgm_vocab_create(data.ctypes.data, off.ctypes.data, 2, None, 0, ctypes.byref(h)) == -1
    off = np.array([0, 1, 2], dtype=np.int64)
    stops = np.array([5], dtype=np.int32)
    assert lib.xgm_vocab_create(data.ctypes.data, off.ctypes.data, 2, stops.ctypes.data, 1, ctypes.byref(h)) == -1
    assert lib.xgm_vocab_create(data.ctypes.data, off.ctypes.data, 0, None, 0, ctypes.byref(h)) == -1
    assert b"" != lib.xgm_last_error()
    assert xgm.bitmask_words(151936) == 4748 and xgm.bitmask_words(33) == 2 and xgm.bitmask_words(0) == 0


# ---------------------------------------------------------------------------
# the GPU kernels' token walk, compiled for the host from the same source
# ---------------------------------------------------------------------------
def _walk_classes_for_nodes(text, root, vocab, nodes=None):
    g = xgm.Grammar(text, root)
    og = oracle.Grammar(text, root)
    toks = vocab.tokens() if hasattr(vocab, "tokens") else vocab.toks
    n_over = 0
    for node in (range(g.num_nodes) if nodes is None else nodes):
        want = og.classify(g.rule_name(g.node_rule(node)), g.node_path(node), vocab)
        for t, w in zip(toks, want):
            got = g.debug_walk_host([node], t, True)
            if got == 3:
                n_over += 1
                got = g.debug_classify_host(node, t)
            assert got == w, (node, g.node_path(node), t, got, int(w))
    return n_over


def test_kernel_walk_classes_match_oracle_arith():
    vocab = si.make_vocab("arith", 1024, 0)
    assert _walk_classes_for_nodes(si.ARITH_GRAMMAR, "expr", vocab) == 0


def test_kernel_walk_classes_match_oracle_json_and_csql_samples():
    vocab = si.make_vocab("bpe", 3000, 2)
    assert _walk_classes_for_nodes(si.JSON_GRAMMAR, "root", vocab, range(0, 74, 3)) == 0
    g = xgm.Grammar(si.CSQL_GRAMMAR, "root")
    rng = np.random.Generator(np.random.PCG64(9))
    nodes = sorted(set(int(n) for n in rng.integers(0, g.num_nodes, size=12)))
    assert _walk_classes_for_nodes(si.CSQL_GRAMMAR, "root", vocab, nodes) == 0


@pytest.mark.parametrize("name", ["arith", "json", "csql", "schema", "xml"])
def test_kernel_walk_masks_match_oracle_along_walks(name):
    """Two-way walk with the full live stack (what the fill kernel runs for
    every stack) OR-ed over the stacks == the oracle's mask, for all tokens."""
    text, root, _ = GRAMMARS[name]
    vocab = si.make_vocab("arith", 1024, 0) if name == "arith" else si.make_vocab("bpe", 4000, 3)
    toks = vocab.tokens()
    first = np.array([t[0] if t else -1 for t in toks], dtype=np.int16)
    g = xgm.Grammar(text, root)
    og = oracle.Grammar(text, root)
    v = xgm.Vocab(vocab.data, vocab.offsets, vocab.stop_ids)
    m = xgm.Matcher(grammar=g, vocab=v)
    om = oracle.EarleyMatcher(og)
    rng = np.random.Generator(np.random.PCG64(zlib.crc32(name.encode()) + 1))
    for step in range(14):
        want = om.mask(vocab)
        stacks = [m.stack(s) for s in range(m.num_stacks())]
        got = np.zeros(len(toks), dtype=bool)
        for i, t in enumerate(toks):
            if not t:
                continue
            for st in stacks:
                r = g.debug_walk_host(st, t, False)
                assert r in (0, 2), (name, st, t, r)
                if r == 2:
                    got[i] = True
                    break
        if m.can_terminate():
            got[vocab.stop_ids] = True
        bad = np.flatnonzero(got != want)
        assert bad.size == 0, (name, step, toks[bad[0]], bool(got[bad[0]]))
        t = si.pick_token(rng, want, first, vocab.stop_ids, structural_bias=0.4)
        if t < 0 or t == int(vocab.stop_ids[0]):
            break
        m.accept_token(t)
        assert om.advance(toks[t])


@pytest.mark.parametrize("name", ["arith", "json", "csql", "schema", "xml"])
def test_frame_below_is_always_a_listed_context(name):
    """Along random walks, the node below every frame of every stack is one of
    the contexts the compiler lists for that frame's rule (the mask cache names
    a stack's token lists by these indices, two frames deep)."""
    text, root, _ = GRAMMARS[name]
    vocab = si.make_vocab("arith", 1024, 0) if name == "arith" else si.make_vocab("bpe", 4000, 3)
    toks = vocab.tokens()
    first = np.array([t[0] if t else -1 for t in toks], dtype=np.int16)
    g = xgm.Grammar(text, root)
    og = oracle.Grammar(text, root)
    v = xgm.Vocab(vocab.data, vocab.offsets, vocab.stop_ids)
    seen = 0
    for seed in range(3):
        m = xgm.Matcher(grammar=g, vocab=v)
        om = oracle.EarleyMatcher(og)
        rng = np.random.Generator(np.random.PCG64(zlib.crc32(name.encode()) + 31 * seed))
        for step in range(40):
            for s in range(m.num_stacks()):
                st = m.stack(s)
                for k in range(len(st) - 1, 0, -1):
                    assert g.debug_context_index(st[k], st[k - 1]) >= 0, (name, seed, step, st, k)
                    seen += 1
            want = om.mask(vocab)
            t = si.pick_token(rng, want, first, vocab.stop_ids, structural_bias=0.4)
            if t < 0 or t == int(vocab.stop_ids[0]):
                break
            m.accept_token(t)
            assert om.advance(toks[t])
    assert seen > 10


def test_kernel_walk_reports_overflow_instead_of_guessing():
    g = xgm.Grammar(si.ARITH_GRAMMAR, "expr")
    start = [n for n in range(g.num_nodes) if g.rule_name(g.node_rule(n)) == "expr" and g.node_path(n) == []][0]
    # every "(" pushes three frames (expr, term, factor): 64 frames are used up
    assert g.debug_walk_host([start], b"(" * 30, True) == 3
    assert g.debug_classify_host(start, b"(" * 30) == 2
    assert g.debug_walk_host([start], b"(" * 15, True) == 2
    assert g.debug_walk_host([start], b"1" * 300, True) == 3     # longer than 255 bytes
    assert g.debug_classify_host(start, b"1" * 300) == 2


def test_vocabulary_size_limit():
    n = 589825
    with pytest.raises(xgm.XgmError) as e:
        xgm.Vocab(np.zeros(1, dtype=np.uint8), np.zeros(n + 1, dtype=np.int64), np.zeros(0, dtype=np.int32))
    assert e.value.args[0] == -10 or "MAX_VOCAB" in str(e.value)


AMBIGUOUS_GRAMMAR = 'root ::= a | b | c\na ::= "a"* "x"\nb ::= "a"* "y" tail\nc ::= ("a" "a")* "z"\ntail ::= "(" root ")" | ""\n'


def _same_state(m1, m2):
    assert m1.is_terminated() == m2.is_terminated()
    if m1.is_terminated():
        return
    s1 = [m1.stack(s) for s in range(m1.num_stacks())]
    s2 = [m2.stack(s) for s in range(m2.num_stacks())]
    assert s1 == s2


@pytest.mark.parametrize("name", ["arith", "json", "csql", "schema", "xml", "ambiguous"])
def test_depth_first_accept_gives_the_engines_stacks(name):
    """The kernels' enumerating depth-first walk over the flattened tables, as a lane does
    it (compiled for the host; the whole-wave form of the accept kernel is compared in
    test_gpu_edges and test_gpu_batch), against the host engine (a breadth-first run of
    the structured automaton): same verdict for every token tried and the same set of
    stacks, in the same order, after every accepted one."""
    if name == "ambiguous":
        text, root = AMBIGUOUS_GRAMMAR, "root"
        vocab = TinyVocab([b"a", b"aa", b"aaa", b"x", b"y", b"z", b"ax", b"aay(", b"(", b")", b"y(a", b"))", b"az", b""], [13])
        toks = vocab.toks
    else:
        text, root, _ = GRAMMARS[name]
        vocab = si.make_vocab("arith", 1024, 0) if name == "arith" else si.make_vocab("bpe", 4000, 3)
        toks = vocab.tokens()
    first = np.array([t[0] if t else -1 for t in toks], dtype=np.int16)
    g = xgm.Grammar(text, root)
    og = oracle.Grammar(text, root)
    v = xgm.Vocab(vocab.data, vocab.offsets, vocab.stop_ids)
    n_ok = n_rejected = n_multi = 0
    for seed in range(20 if name == "ambiguous" else 3):
        m1, m2 = xgm.Matcher(grammar=g, vocab=v), xgm.Matcher(grammar=g, vocab=v)
        om = oracle.EarleyMatcher(og)
        rng = np.random.Generator(np.random.PCG64(zlib.crc32(name.encode()) + 77 * seed))
        for step in range(40):
            want = om.mask(vocab)
            # a few random tokens, allowed or not: same verdict, and a rejection leaves the state alone
            for t in rng.integers(0, len(toks), 6):
                if want[t] or not toks[t]:
                    continue
                assert m1.try_accept_token(int(t)) == -6
                assert m2.debug_try_accept_token_walk(int(t)) == -6
                n_rejected += 1
                _same_state(m1, m2)
            t = si.pick_token(rng, want, first, vocab.stop_ids, structural_bias=0.4)
            if t < 0:
                break
            assert m1.try_accept_token(t) == 0
            assert m2.debug_try_accept_token_walk(t) == 0, (name, seed, step, toks[t])
            _same_state(m1, m2)
            n_ok += 1
            if m1.is_terminated():
                assert m2.debug_try_accept_token_walk(t) == -7
                break
            n_multi += m1.num_stacks() > 1
            assert om.advance(toks[t])
    assert n_ok > 20 and n_rejected > 20, (n_ok, n_rejected)
    if name == "ambiguous":
        assert n_multi > 3


def _random_grammar_text(rng) -> str:
    """A small random grammar over the bytes a-d, '(' and ')': nested groups, repetition, optional parts,
    references (also recursive and in tail position), empty alternatives - the shapes that produce
    parallel stacks, tail calls, shortcuts and returns through several frames."""
    n_rules = int(rng.integers(2, 6))
    names = ["root"] + [f"r{k}" for k in range(1, n_rules)]

    def item(depth):
        u = rng.random()
        if u < 0.40 or depth > 2:
            lit = "".join(rng.choice(list("abcd()")) for _ in range(int(rng.integers(1, 4))))
            return '"' + lit + '"'
        if u < 0.55:
            return "[" + "".join(sorted(set(rng.choice(list("abcd"), size=int(rng.integers(1, 4)))))) + "]"
        if u < 0.80:
            return names[int(rng.integers(0, n_rules))]
        return "( " + alts(depth + 1) + " )"

    def seq(depth):
        parts = []
        for _ in range(int(rng.integers(1, 4))):
            parts.append(item(depth) + rng.choice(["", "", "", "*", "+", "?"]))
        return " ".join(parts)

    def alts(depth):
        k = int(rng.integers(1, 4))
        out = [seq(depth) for _ in range(k)]
        if rng.random() < 0.15:
            out.append('""')
        return " | ".join(out)

    return "\n".join(f"{name} ::= {alts(0)}" for name in names) + "\n"


def test_depth_first_accept_on_random_grammars():
    """Seeded random grammars (those the library accepts: no left recursion, productive root): for random
    byte strings fed a few bytes at a time as tokens, the depth-first accept (the kernels' walk on the host), the
    host engine and the oracle's recogniser agree on every verdict, and the two library routes on the stacks."""
    rng = np.random.Generator(np.random.PCG64(424242))
    pieces = [bytes(p) for p in (b"a", b"b", b"c", b"d", b"(", b")", b"ab", b"ba", b"a(", b")b", b"cd)", b"((", b"))", b"abc", b"dcba", b"(a)")]
    vocab = TinyVocab(pieces + [b""], [len(pieces)])
    n_grammars = n_multi = n_steps = 0
    for trial in range(400):
        text = _random_grammar_text(rng)
        try:
            g = xgm.Grammar(text, "root")
        except xgm.XgmError as e:
            assert e.status in (-4, -5), (text, e)    # left recursion, or nothing derivable
            continue
        og = oracle.Grammar(text, "root")
        v = xgm.Vocab(vocab.data, vocab.offsets, vocab.stop_ids)
        n_grammars += 1
        for walk in range(6):
            m1, m2 = xgm.Matcher(grammar=g, vocab=v), xgm.Matcher(grammar=g, vocab=v)
            prefix = b""
            for step in range(12):
                assert m1.can_terminate() == (og.recognize(prefix) == 2), (text, prefix)
                order = rng.permutation(len(pieces))
                moved = False
                for t in order:
                    rc1 = m1.try_accept_token(int(t))
                    rc2 = m2.debug_try_accept_token_walk(int(t))
                    want = og.recognize(prefix + pieces[t]) > 0
                    if rc1 == -8:          # more than 64 parallel stacks: the engine gives up, state unchanged
                        assert want
                        if rc2 == 0:       # the walk has no such limit: put its matcher back
                            m2 = xgm.Matcher(grammar=g, vocab=v)
                            assert prefix == b"" or m2.try_accept_bytes(prefix) == 0
                            _same_state(m1, m2)
                        continue
                    assert (rc1 == 0) == want, (text, prefix, pieces[t], rc1)
                    assert rc2 == rc1 or (rc2 == -9 and rc1 == 0), (text, prefix, pieces[t], rc1, rc2)
                    if rc2 == -9:          # the walk's limits; take the host's state on both sides
                        m2 = xgm.Matcher(grammar=g, vocab=v)
                        assert m2.try_accept_bytes(prefix + pieces[t]) == 0
                    _same_state(m1, m2)
                    n_steps += 1
                    if rc1 == 0:
                        prefix += pieces[t]
                        n_multi += m1.num_stacks() > 1
                        moved = True
                        break
                if not moved:
                    break
    assert n_grammars > 100 and n_steps > 3000 and n_multi > 100, (n_grammars, n_steps, n_multi)


def _compiled(text, seconds=30.0):
    """The compiled grammar; a compile that does not end fails the test (and is left behind: nothing can stop it)."""
    out = []

    def work():
        try:
            out.append(xgm.Grammar(text, "root"))
        except Exception as e:
            out.append(e)

    thread = threading.Thread(target=work, daemon=True)
    thread.start()
    thread.join(seconds)
    assert out, f"the compile of {text[:100]!r}... ({len(text)} characters) does not end"
    if isinstance(out[0], Exception):
        raise out[0]
    return out[0]


def _letters(n, k=0):
    return "".join(chr(ord("a") + (k + 7 * j + j * j // 26) % 26) for j in range(n))


# Subset construction looks up sets of one NFA state, all that a literal has, by the state and all others by their hash; so
# many of the former come before one of the latter here.  Nodes: one in front of each byte of the literal, and `more`.
@pytest.mark.parametrize("n", [1, 64, 127, 128, 254, 255, 256, 257, 258, 600, 1000, 5000])
@pytest.mark.parametrize("rest, more, good, bad", [
    ("[a-z]*", 1, (b"", b"ab"), (b"1",)),                                          # a loop
    ('ws "}"', 4, (b"}", b"  }"), (b"", b" ")),                                    # a reference that may be skipped
    ('("ab" "x" | "ac" | "a")', 4, (b"abx", b"ac", b"a"), (b"", b"ab", b"acx")),   # alternatives with a common prefix
    ('("=" [0-9]+)?', 3, (b"", b"=12"), (b"=", b"1"))])
def test_literals_of_any_length_compile(n, rest, more, good, bad):
    lit = _letters(n)
    text = f'root ::= "{lit}" {rest}\nws ::= " "*'
    g, og = _compiled(text), oracle.Grammar(text, "root")
    assert g.num_nodes == n + more
    data = lit.encode()
    for tail, ok in [(t, True) for t in good] + [(t, False) for t in bad]:
        m = xgm.Matcher(grammar=g)
        rc = m.try_accept_bytes(data + tail)
        assert (rc == 0) == (og.recognize(data + tail) > 0), tail
        assert (rc == 0 and m.can_terminate()) == ok == (og.recognize(data + tail) == 2), tail
    m = xgm.Matcher(grammar=g)
    if n > 1:
        assert m.try_accept_bytes(data[:-1]) == 0 and not m.can_terminate()
    assert m.try_accept_bytes(b"#") == -6


@pytest.mark.parametrize("n", [2, 15, 16, 17, 18, 40, 60])
def test_alternations_of_names_compile(n):
    names = [_letters(16, 3 * k) + f"{k:02d}" for k in range(n)]
    text = 'root ::= [a-z]* ":" call\ncall ::= (' + " | ".join(f'"{w}"' for w in names) + ') ws "("\nws ::= " "*'
    g, og = _compiled(text), oracle.Grammar(text, "root")
    for data in [f"x:{w}{s}(" for w in names for s in ("", "  ")] + [f":{names[0]}x(", f":{names[-1][:-1]}(", ":("]:
        m = xgm.Matcher(grammar=g)
        assert (m.try_accept_bytes(data.encode()) == 0 and m.can_terminate()) == (og.recognize(data.encode()) == 2), data


@pytest.mark.parametrize("n", [200, 255, 256, 300, 3000])
def test_schemas_with_long_names_compile(n):
    name = _letters(n)
    text = xgm.schema_to_grammar('{"type": "object", "properties": {"%s": {"type": "string"}, "b": {"enum": ["%s", 1]}}}' % (name, name))
    g, og = _compiled(text), oracle.Grammar(text, "root")
    for data in (f'{{"{name}": "x", "b": "{name}"}}', f'{{"{name}":"","b":1}}', f'{{"{name[:-1]}": "x", "b": 1}}', f'{{"{name}": 1, "b": 1}}'):
        m = xgm.Matcher(grammar=g)
        assert (m.try_accept_bytes(data.encode()) == 0 and m.can_terminate()) == (og.recognize(data.encode()) == 2), data[-20:]


# 114 states and 103 nodes a literal: on both sides of 4000 nodes (38, 39: 3991, 4094) and of 8000 states (68, 69: 7957, 8071),
# from where other threads of the compile make what is not in the tables, and take rules in turn, and far beyond.
@pytest.mark.parametrize("n", [20, 37, 38, 39, 68, 69, 76, 80, 300])
def test_grammars_of_many_rules_compile_alike_in_several_threads(n):
    lits = [_letters(97, 5 * k) + f"{k:03d}" for k in range(n)]
    text = si.JSON_GRAMMAR + "\ntop ::= root | " + " | ".join(f'"~" f{k}' for k in range(n)) + "\n"
    text += "\n".join(f'f{k} ::= "{lit}" ("," root)?' for k, lit in enumerate(lits))
    og, made = oracle.Grammar(text, "top"), [None] * 4

    def compile_one(k):
        made[k] = xgm.Grammar(text, "top")

    threads = [threading.Thread(target=compile_one, args=(k,)) for k in range(len(made))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()

    def described(g):
        return [(g.rule_name(g.node_rule(k)), tuple(g.node_path(k))) for k in range(g.num_nodes)]

    assert made[0].num_nodes > 100 * n and all(described(g) == described(made[0]) for g in made[1:])
    for g in made:
        for data in [f"~{lit}{tail}".encode() for lit in (lits[0], lits[n // 2], lits[-1]) for tail in ("", ', {"a": [1e3]}', ",", "x")] + [b"[1, null]", b"~"]:
            m = xgm.Matcher(grammar=g)
            assert (m.try_accept_bytes(data) == 0 and m.can_terminate()) == (og.recognize(data) == 2), data
    # what may follow a rule, and in which contexts: classes of tokens that leave it
    vocab = TinyVocab([b'"', b'a"', b'", ', b'"}', b'"]', b"1}", b"1]", b"},", b"]", b"9", b" ", lits[0][-2:].encode() + b",", b'"~'])
    g = made[-1]
    nodes = [k for k in range(g.num_nodes) if not g.rule_name(g.node_rule(k)).startswith("f") or len(g.node_path(k)) > 99]
    for node in nodes[:: max(1, len(nodes) // 60)]:
        want = og.classify(g.rule_name(g.node_rule(node)), g.node_path(node), vocab)
        assert [g.debug_classify_host(node, t) for t in vocab.toks] == list(want)


@pytest.mark.parametrize("extra, status", [("f0 ::= f0 \"x\" | \"y\"", -4), ("f0 ::= " + " ".join(f'"{"x" * 200}{k}"' for k in range(200)), -9)])
def test_large_grammars_are_refused_as_small_ones_are(extra, status):
    text = "root ::= " + " | ".join(f"f{k}" for k in range(101)) + "\n" + extra + "\n"
    text += "\n".join(f'f{k} ::= "{_letters(100, k)}{k}"' for k in range(1, 101))
    with pytest.raises(xgm.XgmError) as e:
        xgm.Grammar(text, "root")
    assert e.value.status == status


class _ReferenceRules:
    """Minimal automata of rules from their expressions, the long way: positions of the symbols and which can follow which,
    sets of them, states that lead nowhere taken out, the others split until nothing changes.  An expression is ("bytes",
    lo, hi), ("lit", bytes), ("ref", name), ("seq" | "alt", expressions), ("star" | "opt" | "plus", expression); a symbol of
    an automaton a byte or the name of a rule."""

    def __init__(self, rules):
        self.rules = rules
        self.productive = self._least(lambda e, known: self._derives(e, known, True))
        self.nullable = self._least(lambda e, known: self._derives(e, known, False))
        self.automata = {r: self._minimal(*self._sets(e)) for r, e in rules.items() if r in self.productive}

    def _least(self, holds):
        known = set()
        while True:
            more = {r for r, e in self.rules.items() if r not in known and holds(e, known)}
            if not more:
                return known
            known |= more

    def _derives(self, e, known, consumes):
        kind = e[0]
        if kind in ("bytes", "lit"):
            return consumes or (kind == "lit" and not e[1])
        if kind == "ref":
            return e[1] in known
        if kind in ("seq", "alt"):
            return (all if kind == "seq" else any)(self._derives(x, known, consumes) for x in e[1])
        return kind in ("star", "opt") or self._derives(e[1], known, consumes)

    def _sets(self, e):
        """(states, start): a state is (can end, {symbol: state})."""
        symbol, follow = [], []

        def position(s):
            symbol.append(s)
            follow.append(set())
            return len(symbol) - 1

        def parts(e):  # (may be empty, first positions, last positions)
            kind = e[0]
            if kind == "bytes":
                p = position((e[1], e[2]))
                return False, {p}, {p}
            if kind == "ref":
                if e[1] not in self.productive:
                    return False, set(), set()
                p = position(e[1])
                return e[1] in self.nullable, {p}, {p}
            if kind == "lit":
                ps = [position((c, c)) for c in e[1]]
                for p, q in zip(ps, ps[1:]):
                    follow[p].add(q)
                return not ps, set(ps[:1]), set(ps[-1:])
            if kind == "alt":
                xs = [parts(x) for x in e[1]]
                return any(x[0] for x in xs), set().union(*(x[1] for x in xs)), set().union(*(x[2] for x in xs))
            if kind == "seq":
                empty, first, last = True, set(), set()
                for x in e[1]:
                    x_empty, x_first, x_last = parts(x)
                    for p in last:
                        follow[p] |= x_first
                    if empty:
                        first = first | x_first
                    last = last | x_last if x_empty else x_last
                    empty = empty and x_empty
                return empty, first, last
            empty, first, last = parts(e[1])
            if kind != "opt":
                for p in last:
                    follow[p] |= first
            return empty or kind != "plus", first, last

        empty, first, last = parts(e)
        start = (empty, frozenset(first))
        states, work = {}, [start]
        while work:
            s = work.pop()
            if s in states:
                continue
            states[s] = to = {}
            by_symbol = {}
            for p in s[1]:
                for x in [symbol[p]] if isinstance(symbol[p], str) else range(symbol[p][0], symbol[p][1] + 1):
                    by_symbol.setdefault(x, []).append(p)
            for x, ps in by_symbol.items():
                to[x] = (any(p in last for p in ps), frozenset().union(*(follow[p] for p in ps)))
                work.append(to[x])
        return states, start

    @staticmethod
    def _minimal(states, start):
        into = {}
        for s, to in states.items():
            for t in to.values():
                into.setdefault(t, []).append(s)
        alive, work = set(), [s for s in states if s[0]]
        while work:
            s = work.pop()
            if s not in alive:
                alive.add(s)
                work += into.get(s, [])
        block = {s: int(s[0]) for s in alive}
        while True:
            signatures = {s: (block[s], frozenset((x, block[t]) for x, t in states[s].items() if t in alive)) for s in alive}
            numbers = {}
            new = {s: numbers.setdefault(sig, len(numbers)) for s, sig in signatures.items()}
            done = len(numbers) == len(set(block.values()))
            block = new
            if done:
                break
        edges = {block[s]: {x: block[t] for x, t in states[s].items() if t in alive} for s in alive}
        return edges, block[start], {block[s] for s in alive if s[0]}

    def check(self, g):
        """Every rule of the compiled grammar has these states: reached by the same symbols, ending the rule alike."""
        names = [g.rule_name(r) for r in range(g.num_rules)]
        states = {n: {} for n in names}
        for node in range(g.num_nodes):
            name = names[g.node_rule(node)]
            edges, at, final = self.automata[name]
            for x in g.node_path(node):
                at = edges[at][x]
            assert at not in states[name], (name, node, states[name][at])
            states[name][at] = node
            assert g.node_is_final(node) == (at in final), (name, node)
        for n in names:
            assert len(states[n]) == len(self.automata[n][0]), n

    def text(self):
        def show(e):
            kind = e[0]
            if kind == "bytes":
                return f"[{chr(e[1])}-{chr(e[2])}]"
            if kind == "lit":
                return '"' + e[1].decode() + '"'
            if kind == "ref":
                return e[1]
            if kind in ("seq", "alt"):
                return "(" + (" " if kind == "seq" else " | ").join(map(show, e[1])) + ")"
            return "(" + show(e[1]) + ")" + {"star": "*", "opt": "?", "plus": "+"}[kind]
        return "\n".join(f"{r} ::= {show(e)}" for r, e in self.rules.items())


@pytest.mark.parametrize("loops", [False, True])
def test_automata_are_the_minimal_ones(loops):
    """Random rules, with and without loops (those without are minimised from the end, and not at all where no two states
    have equally long ways to an end), against the reference construction; a literal in ten has hundreds of bytes."""
    rng = np.random.Generator(np.random.PCG64(77 + loops))
    n_long = n_merged = n_chain = 0
    for _ in range(150):
        n_rules = int(rng.integers(1, 6))
        names = ["root"] + [f"r{k}" for k in range(1, n_rules)] + ["ws", "dead"]
        rules = {}

        def literal(longest):
            n = int(rng.integers(200, longest)) if rng.random() < 0.1 else int(rng.integers(1, 4))
            return ("lit", bytes(rng.integers(97, 97 + (2 if n < 4 else 26), size=n).astype(np.uint8)))

        def expression(k, depth):
            x = rng.random()
            if depth == 0 or x < 0.3:
                if x < 0.08:
                    lo = int(rng.integers(97, 101))
                    return ("bytes", lo, lo + int(rng.integers(0, 3)))
                if x < 0.25 and k + 1 < len(names):
                    return ("ref", names[int(rng.integers(k + 1, len(names)))])
                return literal(1000 if not loops else 400)
            if x < 0.7:
                return ("seq", [expression(k, depth - 1) for _ in range(int(rng.integers(2, 5)))])
            if x < 0.9 or not loops:
                return ("alt" if x < 0.9 else "opt", [expression(k, depth - 1) for _ in range(int(rng.integers(2, 4)))] if x < 0.9 else expression(k, depth - 1))
            return (str(rng.choice(["star", "plus", "opt"])), expression(k, depth - 1))

        for k in range(n_rules):
            rules[names[k]] = ("seq", [expression(k, 3), ("ref", names[k + 1])]) if k + 1 < n_rules else expression(k, 3)
        rules["ws"] = ("star", ("lit", b" "))
        rules["dead"] = ("seq", [("lit", b"x"), ("ref", "dead")])
        want = _ReferenceRules(rules)
        text = want.text()
        if "root" not in want.productive:
            with pytest.raises(xgm.XgmError) as e:
                xgm.Grammar(text, "root")
            assert e.value.status == -5
            continue
        g = _compiled(text)
        want.check(g)
        n_long += len(text) > 256
        for r in range(g.num_rules):
            edges = want.automata[g.rule_name(r)][0]
            n_merged += len(edges) < len(want._sets(rules[g.rule_name(r)])[0])
            n_chain += len(edges) > 200
    assert n_long > 20 and n_chain > 20 and n_merged > 20, (n_long, n_chain, n_merged)


def test_binding_refuses_what_is_no_number_and_keeps_a_sequence_alive():
    """The calls that csrc/pybinding.cpp marshals take what ctypes and int() take, and no more."""
    v = xgm.Vocab(np.frombuffer(b"123", dtype=np.uint8), np.arange(4, dtype=np.int64), [])
    g = xgm.Grammar('root ::= [0-9]*', "root")
    m = xgm.Matcher(grammar=g, vocab=v)
    for wrong in (None, [], "x1"):
        with pytest.raises((TypeError, ValueError)):
            m.accept_token(wrong)
    m.accept_token(np.int64(1))
    m.accept_token(token_id=2)
    m.accept_bytes(b"7" * 1000)
    with pytest.raises(TypeError):
        m.accept_bytes("7")
    with pytest.raises(TypeError):
        xgm.apply_token_bitmask_inplace(0, None, 1, 1, 1, 0, 1)
    with pytest.raises(TypeError):
        xgm.apply_token_bitmask_inplace(1.5, xgm.DTYPE_F32, 1, 1, 1, 0, 1)
    with pytest.raises(TypeError):
        xgm.fill_and_apply([m], 0, 0, xgm.DTYPE_F32, None, 1)
    # matchers without a cache are refused by the library, also those that only the generator has
    for matchers in ([m], (m,), (xgm.Matcher(grammar=g, vocab=v) for _ in range(300))):
        with pytest.raises(xgm.XgmError) as e:
            xgm.fill_next_token_bitmask(matchers, 64)
        assert e.value.status == -1


@pytest.mark.parametrize("call", ["accept_token", "accept_bytes"])
def test_other_threads_run_while_a_token_is_accepted(call):
    """A token of a megabyte, and a few bytes that each double the number of parallel stacks: another thread goes on
    meanwhile."""
    long_token, doubling = b'"' + b"a" * (1 << 20), b"x" * 15
    v = xgm.Vocab(np.frombuffer(long_token, dtype=np.uint8), np.array([0, len(long_token)], dtype=np.int64), [])
    text = si.JSON_GRAMMAR if call == "accept_token" else 'root ::= a | b\na ::= "x" root? "p"\nb ::= "x" root? "q"'
    m = xgm.Matcher(grammar=xgm.Grammar(text, "root"), vocab=v)
    turns, stop = [0], threading.Event()

    def other():
        while not stop.is_set():
            turns[0] += 1
            time.sleep(1e-4)

    interval = sys.getswitchinterval()
    thread = threading.Thread(target=other)
    try:
        sys.setswitchinterval(100.0)   # the lock changes hands only where it is let go
        thread.start()
        time.sleep(0.01)
        before = turns[0]
        if call == "accept_token":
            m.accept_token(0)
        else:
            with pytest.raises(xgm.XgmError) as e:
                m.accept_bytes(doubling)
            assert e.value.status == -8
        during = turns[0] - before
    finally:
        sys.setswitchinterval(interval)
        stop.set()
        thread.join()
    assert during > 0


def test_the_extension_is_the_one_of_this_python():
    """Its file carries this Python's tag; one without a tag, which any Python would load, is not there."""
    from paper_2411_15100_amd import _native, build
    assert os.path.samefile(_native.__file__, build.EXT)
    assert os.path.basename(build.EXT) == "_native" + sysconfig.get_config_var("EXT_SUFFIX") != "_native.so"
    assert not os.path.exists(build.EXT_UNTAGGED)

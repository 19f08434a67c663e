"""GPU parity at the edges of the kernels' ranges: grammars and sizes where a
level, a tile or a segment begins, ends or is just full.  Expected masks come
from the CPU oracle."""

import numpy as np
import pytest

import oracle
import synth_inputs as si

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

"""The work a user of this library has it do, as measurable cases.

A program that decodes under grammars does five kinds of work with it:

  build      a grammar or a JSON schema arrives: compile it, build its mask cache, take the requests that wait for
             it to where they are, and make their first masks (a new schema per request is the rule in serving, so
             this is on the path of the first token, not only of the start of the program);
  step       one decode step of a batch whose states live on the device: bitmask and masked logits in one launch;
  two_calls  the same step as two calls, as an engine does that masks only some rows of its logits (a row index),
             or whose logits rows are not 16-byte aligned;
  host       whole generations with the states on the host: per step fill and apply, then accept every sampled token;
  draft      speculative decoding with the states on the device: fill and apply before and after every draft token,
             accept it, and go back when the drafts are refused; with `beams` > 1 the rows of a group first take
             over their leader's state (tree decoding).

A case's fields: `kind`; `family` of the grammar (arith, json, csql, script, or schema: random JSON schemas through
the schema front end, `schemas` different ones over the rows from seed `schema` on, string-heavy if `heavy`);
`vocab` tokens; `rows` requests; `dtype` of the logits; `pad` extra logits columns; and what a kind needs besides.

The vocabularies, grammars and the policy by which requests walk through them are those of `synth_inputs`.  Requests
are at random depths of their texts, as in a serving batch; the seed decides where, what they sampled, the logits,
and the names in the schemas of `build`.  All results are exact: masks are bits, and a logit is either kept or -inf.
"""

from __future__ import annotations

import functools
import json
import math

import numpy as np
import torch

import paper_2411_15100_amd as xgm
import synth_inputs as si

LARGEST_VOCAB = 151936
DTYPES = {"f32": (torch.float32, xgm.DTYPE_F32, 4), "bf16": (torch.bfloat16, xgm.DTYPE_BF16, 2),
          "f16": (torch.float16, xgm.DTYPE_F16, 2)}
STRUCTURAL_BIAS = 0.35   # how often a request picks a bracket, quote or comma if it can (synth_inputs.walks)
LONGEST_TEXT = 40        # tokens that a request of a batch has behind it, at most
REJECTED = 0.6           # share of the logits that the masks of schema grammars reject (work() counts their bytes)


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # ---- a decode step in one launch, states on the device
        # an ordinary server, all requests with the same schema
        dict(name="step-schema-48", kind="step", family="schema", schema=0, schemas=1, heavy=False, vocab=128256, rows=48,
             dtype="bf16", pad=0),
        # the serving batch: 128 requests, each with a schema of its own
        dict(name="step-schema-128", kind="step", family="schema", schema=0, schemas=128, heavy=True, vocab=151936, rows=128,
             dtype="bf16", pad=0),
        # ---- fill and apply as two calls
        # an expression grammar over a toy vocabulary: nothing but latency
        dict(name="calls-arith-1", kind="two_calls", family="arith", vocab=1024, rows=1, batch=1, dtype="f32", pad=0),
        # code generation in part of a batch: 24 of 64 logits rows are constrained
        dict(name="rows-csql-24-of-64", kind="two_calls", family="csql", vocab=128256, rows=24, batch=64, dtype="f16", pad=256),
        # an odd vocabulary with unpadded rows: no row but the first is aligned
        dict(name="ragged-json-16", kind="two_calls", family="json", vocab=100003, rows=16, batch=16, dtype="bf16", pad=0),
        # ---- generations with the states on the host
        dict(name="host-json-1", kind="host", family="json", vocab=32000, rows=1, steps=32, form="fused", dtype="f32", pad=0),
        dict(name="host-schema-32", kind="host", family="schema", schema=0, schemas=8, heavy=True, vocab=128256, rows=32, steps=16,
             form="fused", dtype="bf16", pad=0),
        # ---- drafts
        # one local user, JSON mode
        dict(name="draft-json-1", kind="draft", family="json", vocab=32000, rows=1, beams=1, drafts=4, dtype="f32", pad=0),
        # two prompts, four beams each
        dict(name="draft-script-8", kind="draft", family="script", vocab=32000, rows=8, beams=4, drafts=4, dtype="bf16", pad=0),
        dict(name="draft-schema-128", kind="draft", family="schema", schema=0, schemas=32, heavy=True, vocab=151936, rows=128, beams=1,
             drafts=3, dtype="bf16", pad=0),
        # ---- a grammar arrives
        # JSON mode is switched on
        dict(name="build-json", kind="build", family="json", vocab=32000, rows=4),
        # the largest of the schemas, with requests waiting for it
        dict(name="build-schema", kind="build", family="schema", schema=0, schemas=1, heavy=True, vocab=151936, rows=16),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "two_calls", "host", "draft", "build"])
    family = rng.choice(["json", "csql", "script", "schema", "schema", "schema"] + (["arith"] if kind in ("two_calls", "host") else []))
    case = dict(kind=kind, family=family)
    # (the one-launch step of a smaller batch is over before the host can launch the next: see the other kinds for those)
    case["vocab"] = _log_uniform(rng, *((64, 4096) if family == "arith" else (64000 if kind == "step" else 4096, LARGEST_VOCAB)))
    case["rows"] = _log_uniform(rng, *{"step": (48, 128), "two_calls": (1, 128), "host": (1, 32), "draft": (1, 128), "build": (1, 16)}[kind])
    if family == "schema":
        case["schema"] = rng.randrange(1, 16)
        case["schemas"] = 1 if kind == "build" else min(case["rows"], _log_uniform(rng, 1, 16))
        case["heavy"] = rng.random() < 0.7
    if kind != "build":
        case["dtype"] = rng.choice(["bf16", "bf16", "f16", "f32"])
        case["pad"] = rng.choice([0, 0, rng.randrange(1, 513)])
    if kind == "two_calls":
        case["batch"] = case["rows"] if rng.random() < 0.5 else min(128, case["rows"] + _log_uniform(rng, 1, 64))
    if kind == "host":
        case["steps"] = rng.randrange(4, 17)
        case["form"] = rng.choice(["fused", "fused", "static"])
    if kind == "draft":
        case["beams"] = rng.choice([1, 1, 2, 4])
        case["drafts"] = rng.randrange(1, 4)
    return case


def _logits_columns(case):
    """Columns of a logits row.  The fused calls want 16-byte rows, and engines pad their rows anyway."""
    n = case["vocab"] + case["pad"]
    return n if case["kind"] == "two_calls" else -(-n // 64) * 64


def work(case):
    """Masks written, rejected logits written (none has to be read); between two calls the mask is read again.  A
    build reads the vocabulary's tokens and writes the masks it was made for."""
    mask = 4 * -(-case["vocab"] // 32) * case["rows"]
    if case["kind"] == "build":
        return {"bytes": 16 * case["vocab"] + mask, "flops": 0}
    logits = REJECTED * DTYPES[case["dtype"]][2] * _logits_columns(case) * case["rows"]
    if case["kind"] == "two_calls":
        return {"bytes": 2 * mask + logits, "flops": 0}
    return {"bytes": (mask + logits) * {"step": 1, "host": case.get("steps"), "draft": case.get("drafts", 0) + 1}[case["kind"]], "flops": 0}


def tolerance(case):
    return "exact"


# ------------------------------------------------------------------------------- what a program keeps
def _stream():
    return int(torch.cuda.current_stream().cuda_stream)


@functools.lru_cache(maxsize=8)
def _vocabulary(family, size):
    """(handle, starts with a structural byte [size] bool, stop id): the largest vocabulary, or a part of it of the
    wanted size with all single bytes."""
    if family == "arith":
        v = si.make_vocab("arith", size, 0)
        data, offsets, stop = v.data, v.offsets, int(v.stop_ids[0])
    else:
        v = si.make_vocab("bpe", LARGEST_VOCAB, 0)
        lens = np.diff(v.offsets)
        rng = np.random.Generator(np.random.PCG64(size))
        must = np.flatnonzero(lens <= 1)
        rest = rng.permutation(np.flatnonzero(lens > 1))[: size - must.size]
        ids = np.arange(LARGEST_VOCAB) if size == LARGEST_VOCAB else rng.permutation(np.concatenate([must, rest]))
        lens = lens[ids]
        offsets = np.concatenate([[0], np.cumsum(lens)])
        data = v.data[np.repeat(v.offsets[:-1][ids] - offsets[:-1], lens) + np.arange(offsets[-1])]
        stop = int(np.flatnonzero(ids == v.stop_ids[0])[0])
    first = np.zeros(size, dtype=np.uint8)
    some = np.diff(offsets) > 0
    first[some] = data[offsets[:-1][some]]
    structural = torch.from_numpy(np.isin(first, np.fromiter(si.STRUCTURAL_BYTES, dtype=np.uint8)) & some).cuda()
    return xgm.Vocab(data, offsets, [stop]), structural, stop


def _json_schema(node, rename):
    """synth_inputs.random_schema's dict as a JSON schema, its names spelled through `rename`."""
    t = node["type"]
    if t == "enum":
        return {"enum": [v.translate(rename) for v in node["values"]]}
    if t == "array":
        return {"type": "array", "items": _json_schema(node["items"], rename)}
    if t == "object":
        return {"type": "object", "properties": {k.translate(rename): _json_schema(v, rename) for k, v in node["properties"]}}
    return {"type": t}


def _schema_text(seed, heavy, names=None):
    """JSON text of a random schema; `names` (a generator) respells its names by a permutation of the letters, which
    gives another schema of the same size."""
    letters = "abcdefghijklmnopqrstuvwxyz"
    rename = str.maketrans(letters, "".join(names.permutation(list(letters)))) if names is not None else {}
    return json.dumps(_json_schema(si.random_schema(seed, string_heavy=heavy), rename))


@functools.lru_cache(maxsize=256)
def _schema_grammar(seed, heavy):
    return xgm.schema_to_grammar(_schema_text(seed, heavy)), "root"


_FIXED = {"arith": (si.ARITH_GRAMMAR, "expr"), "json": (si.JSON_GRAMMAR, "root"), "csql": (si.CSQL_GRAMMAR, "root"),
          "script": (si.PYDSL_GRAMMAR, "root")}


@functools.lru_cache(maxsize=256)
def _grammar(text, root):
    return xgm.Grammar(text, root)


@functools.lru_cache(maxsize=256)
def _cache(text, root, vocab):
    return xgm.Cache(_grammar(text, root), vocab, _stream())


def _caches(case, vocab, group=1):
    """One mask cache per row (rows of a group of `group` share theirs)."""
    if case["family"] != "schema":
        return [_cache(*_FIXED[case["family"]], vocab)] * case["rows"]
    kinds = [_cache(*_schema_grammar(case["schema"] + k, case["heavy"]), vocab) for k in range(case["schemas"])]
    return [kinds[b // group % case["schemas"]] for b in range(case["rows"])]


# --------------------------------------------------------------------------------------- what requests do
def _walk(batch, rows, family, vocab, gen, lengths):
    """Let every row of a device batch sample `lengths[row]` tokens that its masks allow; a row that has ended stays.
    Returns the tokens, int32 [steps, rows] on the device, -1 where a row sat out."""
    handle, structural, stop = vocab
    V = handle.size
    mask = torch.zeros((rows, xgm.bitmask_words(V)), dtype=torch.int32, device="cuda")
    shifts = torch.arange(32, dtype=torch.int32, device="cuda")
    lengths = torch.as_tensor(lengths, device="cuda")
    done = torch.zeros(rows, dtype=torch.bool, device="cuda")
    tokens = []
    for t in range(int(lengths.max())):
        batch.fill_next_token_bitmask(mask.data_ptr(), _stream())
        allowed = ((mask.unsqueeze(2) >> shifts) & 1).view(rows, -1)[:, :V]
        score = torch.randint(1, 1 << 62, (rows, V), generator=gen, device="cuda") * allowed
        score[:, stop] = 0
        best, pick = score.max(1)
        if family != "arith":
            s_best, s_pick = (score * structural).max(1)
            biased = (torch.rand(rows, generator=gen, device="cuda") < STRUCTURAL_BIAS) & (s_best > 0)
            pick = torch.where(biased, s_pick, pick)
        pick = torch.where(best > 0, pick, stop)
        pick = torch.where((t < lengths) & ~done, pick, -1).to(torch.int32)
        batch.accept_tokens(pick.data_ptr(), _stream())
        refused = torch.from_numpy(batch.status(_stream()) != 0).cuda()  # a state beyond the device's limits: the row stays
        tokens.append(torch.where(refused, -1, pick))
        done |= refused | (pick == stop)
    return torch.stack(tokens) if tokens else torch.empty((0, rows), dtype=torch.int32, device="cuda")


def _logits(case, gen, rows, buffers=None):
    dtype = DTYPES[case["dtype"]][0]
    shape = (rows, _logits_columns(case))
    if buffers is None:
        return torch.randn(shape, generator=gen, device="cuda").to(dtype)
    out = torch.empty((buffers,) + shape, dtype=dtype, device="cuda")
    for k in range(buffers):
        out[k] = torch.randn(shape, generator=gen, device="cuda")
    return out


class _State:
    """Inputs of one case; `run` is what a program does with them."""

    def __init__(self, case, seed):
        self.stream = _stream()
        self.vocab = _vocabulary("arith" if case["family"] == "arith" else "bpe", case["vocab"])
        self.V = case["vocab"]
        self.rows = case["rows"]
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        self.rng = np.random.Generator(np.random.PCG64(seed))
        self.mask = torch.zeros((self.rows, xgm.bitmask_words(self.V)), dtype=torch.int32, device="cuda")
        if case["kind"] != "build":
            self.dtype = DTYPES[case["dtype"]][1]
            self.columns = _logits_columns(case)

    def started(self, case, caches, history):
        """A device batch whose rows are 0 to LONGEST_TEXT tokens into their texts."""
        batch = xgm.DeviceBatch([xgm.Matcher(cache=c) for c in caches], history=history, stream=self.stream)
        _walk(batch, self.rows, case["family"], self.vocab, self.gen, self.rng.integers(0, LONGEST_TEXT + 1, size=self.rows))
        return batch


class _Step(_State):
    def __init__(self, case, seed):
        super().__init__(case, seed)
        self.batch = self.started(case, _caches(case, self.vocab[0]), history=0)
        self.logits = _logits(case, self.gen, self.rows)

    def run(self):
        self.batch.fill_and_apply(self.mask.data_ptr(), self.logits.data_ptr(), self.dtype, self.columns, self.columns,
                                  stream=self.stream)
        return self.mask, self.logits


class _TwoCalls(_State):
    def __init__(self, case, seed):
        super().__init__(case, seed)
        self.batch = self.started(case, _caches(case, self.vocab[0]), history=0)
        self.total = case["batch"]
        self.logits = _logits(case, self.gen, self.total)
        # the constrained rows among those of the logits
        self.index = None
        if self.total > self.rows:
            self.index = torch.from_numpy(self.rng.permutation(self.total)[: self.rows].astype(np.int32)).cuda()

    def run(self):
        self.batch.fill_next_token_bitmask(self.mask.data_ptr(), self.stream)
        xgm.apply_token_bitmask_inplace(self.logits.data_ptr(), self.dtype, self.total, self.columns, self.columns,
                                        self.mask.data_ptr(), self.V, 0 if self.index is None else self.index.data_ptr(),
                                        self.rows, stream=self.stream)
        return self.mask, self.logits


class _Host(_State):
    def __init__(self, case, seed):
        super().__init__(case, seed)
        caches = _caches(case, self.vocab[0])
        self.matchers = [xgm.Matcher(cache=c) for c in caches]
        self.together = xgm.MatcherBatch(self.matchers)
        self.fused = case["form"] == "fused"
        scout = xgm.DeviceBatch(self.matchers, history=0, stream=self.stream)
        self.tokens = _walk(scout, self.rows, case["family"], self.vocab, self.gen, np.full(self.rows, case["steps"])).tolist()
        self.logits = _logits(case, self.gen, self.rows, case["steps"])  # one buffer per step: what a model would write

    def run(self):
        for m in self.matchers:
            m.reset()
        for logits, tokens in zip(self.logits, self.tokens):
            if self.fused:
                xgm.fill_and_apply(self.together, self.mask.data_ptr(), logits.data_ptr(), self.dtype, self.columns, self.columns,
                                   stream=self.stream)
            else:
                xgm.fill_next_token_bitmask_static(self.matchers, self.mask.data_ptr(), self.stream)
                xgm.apply_token_bitmask_inplace(logits.data_ptr(), self.dtype, self.rows, self.columns, self.columns,
                                                self.mask.data_ptr(), self.V, stream=self.stream)
            for m, t in zip(self.matchers, tokens):
                if t >= 0:
                    m.accept_token(t)
        return self.mask, self.logits


class _Draft(_State):
    def __init__(self, case, seed):
        super().__init__(case, seed)
        beams, drafts = case["beams"], case["drafts"]
        self.batch = self.started(case, _caches(case, self.vocab[0], beams), history=drafts + 1)
        rows = torch.arange(self.rows, dtype=torch.int32, device="cuda")
        self.leaders = rows // beams * beams if beams > 1 else None
        if self.leaders is not None:
            self.batch.fork(self.leaders.data_ptr(), self.stream)
        # rows get between one draft token and all of them
        self.tokens = _walk(self.batch, self.rows, case["family"], self.vocab, self.gen,
                            self.rng.integers(1, drafts + 1, size=self.rows) if self.rows > 1 else np.array([drafts]))
        self.back = (self.tokens >= 0).sum(0).to(torch.int32)
        if self.leaders is not None:
            self.back += (self.leaders != rows).to(torch.int32)
        self.batch.rollback(self.back.data_ptr(), self.stream)
        self.logits = _logits(case, self.gen, self.rows, len(self.tokens) + 1)

    def run(self):
        if self.leaders is not None:
            self.batch.fork(self.leaders.data_ptr(), self.stream)
        for k, logits in enumerate(self.logits):
            if k:
                self.batch.accept_tokens(self.tokens[k - 1].data_ptr(), self.stream)
            self.batch.fill_and_apply(self.mask.data_ptr(), logits.data_ptr(), self.dtype, self.columns, self.columns,
                                      stream=self.stream)
        self.batch.rollback(self.back.data_ptr(), self.stream)
        return self.mask, self.logits


class _Build(_State):
    def __init__(self, case, seed):
        super().__init__(case, seed)
        self.schema = _schema_text(case["schema"], case["heavy"], self.rng) if case["family"] == "schema" else None
        text, root = (xgm.schema_to_grammar(self.schema), "root") if self.schema else _FIXED[case["family"]]
        cache = xgm.Cache(xgm.Grammar(text, root), self.vocab[0], self.stream)
        scout = xgm.DeviceBatch([xgm.Matcher(cache=cache)] * self.rows, history=0, stream=self.stream)
        tokens = _walk(scout, self.rows, case["family"], self.vocab, self.gen, self.rng.integers(0, 25, size=self.rows))
        self.texts = [[t for t in row if t >= 0] for row in tokens.T.tolist()]
        self.text, self.root = text, root

    def run(self):
        text = self.text if self.schema is None else xgm.schema_to_grammar(self.schema)
        cache = xgm.Cache(xgm.Grammar(text, self.root), self.vocab[0], self.stream)
        matchers = [xgm.Matcher(cache=cache) for _ in range(self.rows)]
        for m, tokens in zip(matchers, self.texts):
            for t in tokens:
                m.accept_token(t)
        xgm.fill_next_token_bitmask(matchers, self.mask.data_ptr(), self.stream)
        return self.mask


_KINDS = {"step": _Step, "two_calls": _TwoCalls, "host": _Host, "draft": _Draft, "build": _Build}


def prepare(case, seed):
    return _KINDS[case["kind"]](case, seed)


def run(state):
    return state.run()

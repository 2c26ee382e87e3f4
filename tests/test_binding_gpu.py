"""The binding's native marshalling against its Python code: the same results
for the arguments it takes, and nothing accepted that the Python code refuses."""
import types

import numpy as np
import pytest
import torch

import paper_2608_03447_amd as asd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class _Declines:
    """A native module that takes no call."""
    def __getattr__(self, name):
        return lambda *args: None


class _Counts:
    """The native module, counting the calls it takes."""
    def __init__(self, fast):
        self.fast, self.taken = fast, 0

    def __getattr__(self, name):
        def call(*args):
            r = getattr(self.fast, name)(*args)
            self.taken += r is not None
            return r
        return call


def _state(dtype=torch.bfloat16, vocab=1000, n=5, k=3):
    gen = torch.Generator(device=DEV).manual_seed(7)
    rows = n * (k + 1)
    s = types.SimpleNamespace(rows=rows, vocab=vocab, n=n)
    s.logits = torch.randn((rows, vocab), generator=gen, device=DEV).to(dtype)
    s.draft = s.logits.float().argmax(1).to(torch.int32)
    s.draft[::3] = 5
    s.lens = torch.full((n,), k, dtype=torch.int32, device=DEV)
    s.tau = torch.full((n,), 2.0, device=DEV)
    s.cap = torch.full((n,), 1, dtype=torch.int32, device=DEV)
    s.budget = torch.tensor([[8.0, 0.0]] * n, device=DEV)
    s.offsets = torch.arange(n, device=DEV) * (k + 1)
    s.argmax = torch.empty(rows, dtype=torch.int32, device=DEV)
    s.regret = torch.empty(rows, dtype=torch.float32, device=DEV)
    s.hidden = torch.randn((rows, 128), generator=gen, device=DEV).to(torch.bfloat16)
    s.weight = torch.randn((vocab, 128), generator=gen, device=DEV).to(torch.bfloat16)
    s.tokens = torch.zeros((n, 64), dtype=torch.int32, device=DEV)
    s.seq = torch.zeros(n, dtype=torch.int64, device=DEV)
    s.partials = torch.empty((1, rows, 4), dtype=torch.int32, device=DEV)
    s.counts = torch.zeros((2, 2), dtype=torch.int64, device=DEV)
    s.mism = torch.zeros(1, dtype=torch.int64, device=DEV)
    s.taus = torch.tensor([0.5, 4.0], device=DEV)
    s.ps = torch.tensor([0, 1], dtype=torch.int32, device=DEV)
    return s


def _rest(s):
    return s.draft, s.lens, s.tau, s.cap, s.budget


CALLS = {
    "verify": lambda s: asd.asd_verify(s.logits, *_rest(s), out_argmax=s.argmax, out_regret=s.regret),
    "static": lambda s: asd.asd_verify_static(s.logits, *_rest(s), row_offsets=s.offsets),
    "raw": lambda s: asd.asd_verify_ex(s.logits, *_rest(s), flags=asd.ASD_GATE_RAW),
    "commit": lambda s: asd.asd_verify_commit(s.logits, *_rest(s), s.tokens, s.seq),
    "shard": lambda s: (asd.asd_shard_argmax(s.logits, 0, s.vocab, s.draft, s.partials[0]),
                        *asd.asd_verify_partials(s.partials, s.vocab, s.vocab, *_rest(s))),
    "lmhead": lambda s: asd.asd_lmhead_verify(s.hidden, s.weight, *_rest(s), out_argmax=s.argmax,
                                              out_regret=s.regret),
    "opportunity": lambda s: (asd.asd_verify(s.logits, *_rest(s), out_argmax=s.argmax,
                                             out_regret=s.regret),
                              asd.asd_opportunity(s.draft, s.argmax, s.regret, s.vocab, s.lens,
                                                  s.taus, s.ps, s.counts, s.mism))[0],
}


def _outputs(s, call):
    out = list(CALLS[call](s)) + [s.budget, s.tokens, s.seq, s.counts, s.mism]
    if call in ("verify", "lmhead", "opportunity"):
        out += [s.argmax, s.regret]
    torch.cuda.synchronize()
    return [t.cpu().numpy().view(np.int32) for t in out]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("call", sorted(CALLS))
def test_native_calls_equal_python_calls(call, dtype, monkeypatch):
    counts = _Counts(asd._load_fast())
    monkeypatch.setattr(asd, "_fast", counts)
    native = _outputs(_state(dtype), call)
    assert counts.taken == (2 if call in ("shard", "opportunity") else 1)
    monkeypatch.setattr(asd, "_fast", _Declines())
    python = _outputs(_state(dtype), call)
    for a, b in zip(native, python):
        assert np.array_equal(a, b)


def test_calls_run_without_a_binding(monkeypatch):
    native = _outputs(_state(), "verify")
    monkeypatch.setattr(asd, "_fast", None)
    monkeypatch.setattr(asd, "BINDING", asd.BINDING + ".missing")
    with pytest.warns(RuntimeWarning, match="Python marshalling"):
        python = _outputs(_state(), "verify")
    for a, b in zip(native, python):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("n", [0, 2])
def test_given_outputs_are_the_ones_returned(n, native, monkeypatch):
    monkeypatch.setattr(asd, "_fast", asd._load_fast() if native else _Declines())
    s = _state(n=max(n, 1), k=1)
    acc = torch.empty(n, dtype=torch.int32, device=DEV)
    nxt = torch.empty(n, dtype=torch.int32, device=DEV)
    rows = 2 * n
    out = asd.asd_verify(s.logits[:rows], s.draft[:rows], s.lens[:n], s.tau[:n], s.cap[:n],
                         s.budget[:n], out_accept_len=acc, out_next_token=nxt)
    assert out[0] is acc and out[1] is nxt


CHANGES = {
    "scalar controls": lambda s: setattr(s, "tau", 2.0) or setattr(s, "cap", 1),
    "strided drafts": lambda s: setattr(s, "draft", s.draft.repeat_interleave(2)[::2]),
    "strided lengths": lambda s: setattr(s, "lens", s.lens.repeat_interleave(2)[::2]),
    "strided logits": lambda s: setattr(s, "logits", s.logits.t().contiguous().t()),
    "half logits": lambda s: setattr(s, "logits", s.logits.half()),
    "logits on the host": lambda s: setattr(s, "logits", s.logits.cpu()),
    "one draft too few": lambda s: setattr(s, "draft", s.draft[:-1].contiguous()),
    "long drafts": lambda s: setattr(s, "draft", s.draft.long()),
    "lengths on the host": lambda s: setattr(s, "lens", s.lens.cpu()),
    "double gates": lambda s: setattr(s, "tau", s.tau.double()),
    "one cap too many": lambda s: setattr(s, "cap", s.cap.repeat(2)),
    "flat ledgers": lambda s: setattr(s, "budget", s.budget.flatten()),
    "strided ledgers": lambda s: setattr(s, "budget", s.budget.t().contiguous().t()),
    "short argmax": lambda s: setattr(s, "argmax", s.argmax[:-1]),
    "long regret": lambda s: setattr(s, "regret", s.regret.long()),
}


@pytest.mark.parametrize("change", sorted(CHANGES))
def test_other_arguments_are_left_to_python(change, monkeypatch):
    """The native function declines them: converted or refused as before."""
    results = []
    for fast in (_Counts(asd._load_fast()), _Declines()):
        monkeypatch.setattr(asd, "_fast", fast)
        s = _state()
        CHANGES[change](s)
        try:
            results.append(_outputs(s, "verify"))
        except ValueError as e:
            results.append(str(e))
        if isinstance(fast, _Counts):
            assert fast.taken == 0
    if isinstance(results[0], str) or isinstance(results[1], str):
        assert results[0] == results[1]
    else:
        assert all(np.array_equal(a, b) for a, b in zip(*results))


def test_failing_status_raises():
    s = _state()
    with pytest.raises(asd.AsdError) as e:
        asd.asd_lmhead_verify(s.hidden[:, :64].contiguous(), s.weight[:, :64].contiguous(), *_rest(s))
    assert e.value.status == 1          # d is not a multiple of 128

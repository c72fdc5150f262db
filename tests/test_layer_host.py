"""Host-side bookkeeping of the layer object (no GPU): the transposed copies of the
private expert weights that the backward uses are made once, kept across backward
calls, and remade after an optimizer step, an in-place torch update or new tensors. A step
of the layer that was replaced, wherever, is the one that a forward calls."""
import types

import pytest
import torch

import paper_2608_06690_amd as P
from paper_2608_06690_amd import _native as N
from paper_2608_06690_amd import layer as Lmod


def make_layer():
    H, I, npub, npriv = 16, 8, 3, 2
    desc = P.make_desc(H, 64, npub, npriv, 2)
    w = lambda *s: torch.randn(*s)  # noqa: E731
    return Lmod.PolicyMaskedMoE(desc, w(npub, H), w(npriv, H), None, w(npub, 2 * I, H), w(npub, H, I),
                                w(npriv, 2 * I, H), w(npriv, H, I))


def test_private_transposes_made_once_and_after_changes(monkeypatch):
    calls = []

    def transpose(src, dst, stream=None):
        calls.append(src.data_ptr())
        dst.copy_(src.transpose(1, 2))

    monkeypatch.setattr(N, "pmpe_transpose_experts", transpose)
    monkeypatch.setattr(N, "pmpe_adamw", lambda *a, **k: None)
    lay = make_layer()
    wt = lay.transposed_weights()
    assert len(calls) == 4  # public W2, W13 once; private W2, W13
    assert torch.equal(wt[2], lay.w2_priv.transpose(1, 2)) and torch.equal(wt[3], lay.w13_priv.transpose(1, 2))
    calls.clear()
    lay.transposed_weights()
    lay.transposed_weights()
    assert calls == []  # kept across backward calls
    # an in-place torch update of a private weight is seen through its version counter
    lay.w2_priv.mul_(2.0)
    wt = lay.transposed_weights()
    assert len(calls) == 2 and torch.equal(wt[2], lay.w2_priv.transpose(1, 2))
    calls.clear()
    # the optimizer step remakes them once (its kernel writes through a raw pointer)
    g = Lmod.GradBuffers(None, torch.zeros_like(lay.w13_priv), torch.zeros_like(lay.w2_priv),
                         torch.zeros_like(lay.wr_priv), None, None)
    opt = P.PrivateAdamW(lay)
    opt.step(g)
    assert len(calls) == 2
    calls.clear()
    lay.transposed_weights()
    assert calls == []
    # new private tensors
    lay.w13_priv = torch.randn_like(lay.w13_priv)
    wt = lay.transposed_weights()
    assert len(calls) == 2 and torch.equal(wt[3], lay.w13_priv.transpose(1, 2))
    # the public copies are never remade
    assert all(c not in calls for c in (lay.w2_pub.data_ptr(), lay.w13_pub.data_ptr()))


STEPS = ["route", "dispatch", "expert_ffn", "combine", "audit"]
CALLS = ["pmpe_route", "pmpe_dispatch", "pmpe_expert_ffn", "pmpe_combine", "pmpe_audit"]


@pytest.mark.parametrize("where", ["nowhere", "subclass", "object", "class", "binding"])
@pytest.mark.parametrize("step", range(5))
def test_a_replaced_step_is_called(monkeypatch, where, step):
    seen = []
    monkeypatch.setattr(Lmod.PolicyMaskedMoE, "buffers", lambda self, T: None)
    monkeypatch.setattr(Lmod.PolicyMaskedMoE, "_forward", lambda self, *a, **k: seen.append("one call"))

    def step_of(name):
        return lambda *a, **k: seen.append(name)

    lay = make_layer()
    if where == "subclass":
        lay.__class__ = type("Traced", (Lmod.PolicyMaskedMoE,), {n: step_of(n) for n in STEPS})
    elif where == "object":
        lay.__dict__.update({n: step_of(n) for n in STEPS})
    elif where == "class":
        monkeypatch.setattr(Lmod.PolicyMaskedMoE, STEPS[step], step_of(STEPS[step]))
    elif where == "binding":
        monkeypatch.setattr(N, CALLS[step], step_of(CALLS[step]))
    assert lay._plain_steps() == (where == "nowhere")
    if where in ("nowhere", "subclass", "object"):
        lay.forward(torch.zeros(4, 16), None, None, torch.tensor([0, 4]))
        assert seen == (["one call"] if where == "nowhere" else STEPS)


@pytest.mark.parametrize("offsets", [None, torch.tensor([0, 4], dtype=torch.int32)])
@pytest.mark.parametrize("fp8", [False, True])
def test_arguments_of_the_one_call(monkeypatch, offsets, fp8):
    """A forward without requests needs the counters of its audit argument only, and any iterable of eight
    fp8 tensors will do."""
    got = []
    monkeypatch.setattr(N, "pmpe_layer_forward", lambda d, T, tensors, R, ffn, stream: got.extend((tensors, R, ffn)))
    lay = make_layer()
    b = types.SimpleNamespace(**{f: torch.zeros(1) for f in Lmod.LayerBuffers.__dataclass_fields__})
    monkeypatch.setattr(Lmod.PolicyMaskedMoE, "buffers", lambda self, T: b)
    counters = dict(token_rows=torch.zeros(4), priv_calls=torch.zeros(2))
    reduce = dict(req_rows=torch.zeros(1), total=torch.zeros(1), violations=torch.zeros(1))
    audit = types.SimpleNamespace(**counters, **({} if offsets is None else reduce))
    x = torch.zeros(4, 16)
    if fp8:
        weights = {i: torch.zeros(1) for i in range(8)}
        lay.forward_fp8(x, None, weights.values(), audit, offsets)
    else:
        lay.forward(x, None, audit, offsets)
    arg = dict(zip(N.ForwardArgs.POINTERS, got[0]))
    assert len(got[0]) == len(N.ForwardArgs.POINTERS) and got[1] == (0 if offsets is None else 1)
    assert arg["req_offset"] is offsets and arg["audit_token_rows"] is counters["token_rows"]
    for name, field in (("req_private_rows", "req_rows"), ("total_private_rows", "total"), ("deny_violations", "violations")):
        assert arg[name] is (None if offsets is None else reduce[field])
    if fp8:
        assert arg["w13_pub"] is weights[0] and arg["w2s_priv"] is weights[7] and arg["w13_sh"] is None

"""The native half of the binding takes the usual arguments only: anything else comes back undone, and the checks one by one say
what is wrong or take it after all."""
import pytest
import torch

from paper_2404_19124_amd import binding as B

I32 = dict(dtype=torch.int32)


def _verify(dev, b=3, Bc=4, n=2, V=70, dtype=torch.float32):
    g = torch.Generator().manual_seed(5)
    logits = torch.randn((b, Bc, n + 1, V), generator=g).to(dtype).to(dev)
    cand = torch.randint(0, V, (b, Bc, n), generator=g, dtype=torch.int32).to(dev)
    outs = [torch.full(s, -7, device=dev, **I32) for s in ((b, Bc, n + 1), (b,), (b,), (b, n + 1), (b,), (b, Bc))]
    return logits, cand, outs


def test_nothing_happens_on_host_tensors():
    logits, cand, outs = _verify("cpu")
    f = B._native()
    assert f.verify(logits, cand, None, *outs, None) is None
    assert f.verify(logits, cand, None, *outs) is None                    # an argument is missing
    assert f.verify(None, cand, None, *outs, None) is None
    hidden = torch.zeros((3, 4, 3, 8))
    assert f.advance(hidden, outs[1], outs[2], outs[3], torch.zeros((3, 8)), outs[4], None) is None
    assert f.tree_metadata(cand, *outs, None, None) is None
    for handle, top_k, Bc in ((None, (2, 1), 2), (0, (2.0, 1), 2), (0, (2, 1), 2.0), (0, "21", 2), (0, (2, 1), 1 << 70)):
        assert f.draft(handle, 2, 64, B.SPEC_BF16, torch.zeros((3, 64)), outs[1], top_k, Bc, cand, torch.zeros((3, 4)), outs[5], None) is None
    assert all((o == -7).all() for o in outs)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("dynamic", [False, True])
def test_both_ways_agree(monkeypatch, dtype, dynamic):
    logits, cand, outs = _verify("cuda", dtype=dtype)
    n_cand = torch.tensor([4, 0, 2], device="cuda", **I32)
    call = (lambda x, o: B.spec_verify_dynamic(x, cand, n_cand, *o)) if dynamic else (lambda x, o: B.spec_verify(x, cand, *o))
    assert B._native().verify(logits, cand, n_cand if dynamic else None, *outs, None) == B.SPEC_OK
    want = [o.clone() for o in outs]
    for x in (logits, torch.nn.Parameter(logits)):   # a subclass goes the other way
        got = [torch.full_like(o, -7) for o in outs]
        call(x, got)
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    hidden = torch.randn((3, 4, 3, 8), device="cuda").to(dtype)
    state, tok = torch.zeros((2, 3, 8), device="cuda", dtype=dtype), torch.zeros((2, 3), device="cuda", **I32)
    B.spec_advance(hidden, want[2], want[1], want[3], state[0], tok[0])
    B.spec_advance(torch.nn.Parameter(hidden), want[2], want[1], want[3], state[1], tok[1])
    assert torch.equal(state[0], state[1]) and torch.equal(tok[0], tok[1])


@pytest.mark.gpu
def test_unusual_arguments_are_refused_as_before():
    logits, cand, outs = _verify("cuda")
    with pytest.raises(ValueError, match="greedy must have shape"):
        B.spec_verify(logits, cand, outs[0][:, :3], *outs[1:])
    with pytest.raises(ValueError, match="cand_tokens must have dtype"):
        B.spec_verify(logits, cand.long(), *outs)
    with pytest.raises(ValueError, match="base_logits must be contiguous"):
        B.spec_verify(logits.transpose(0, 1).contiguous().transpose(0, 1), cand, *outs)
    with pytest.raises(ValueError, match="accept_len must be a device tensor"):
        B.spec_verify(logits, cand, outs[0], outs[1].cpu(), *outs[2:])
    with pytest.raises(ValueError, match="n_cand is required"):
        B.spec_verify_dynamic(logits, cand, None, *outs)
    with pytest.raises(AttributeError):
        B.spec_verify(logits, cand, *outs, stream="none")
    with pytest.raises(B.SpecError):   # what the library refuses
        B.spec_verify(logits[:, :, :1].contiguous(), cand[:, :, :0].contiguous(), outs[0][:, :, :1].contiguous(), outs[1], outs[2],
                      outs[3][:, :1].contiguous(), outs[4], outs[5])

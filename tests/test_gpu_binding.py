"""The binding's native half: what it refuses, with which exception, and the gradient buffers it allocates."""
import numpy as np
import pytest
import torch

from paper_2503_06671_amd import binding

pytestmark = pytest.mark.gpu

CA, KS = 4, 3


def call(**change):
    a = dict(x=torch.randn(1, 6, 9, 8, device="cuda"), Ca=CA, lk=torch.randn(CA, KS, KS, device="cuda"),
             workspace=binding.new_workspace(1, CA, 9, 8))
    a.update(change)
    return binding.convattn_forward(**a)


@pytest.mark.parametrize("error, change", [
    (TypeError, lambda: dict(x=torch.randn(1, 6, 9, 8, device="cuda", dtype=torch.float16))),
    (TypeError, lambda: dict(x=torch.randn(1, 6, 8, 9, device="cuda").transpose(2, 3))),
    (TypeError, lambda: dict(lk=torch.randn(CA, KS, KS))),
    (ValueError, lambda: dict(lk=torch.randn(CA + 1, KS, KS, device="cuda"))),
    (ValueError, lambda: dict(lk=torch.randn(8, device="cuda"), ks=3, lk_channel_stride=9)),
    (ValueError, lambda: dict(lk=torch.randn(36, device="cuda"), ks=3, lk_channel_stride=2 ** 64 // 3)),  # three times that is -1 in 64 bits
    (ValueError, lambda: dict(ks=3)),
    (ValueError, lambda: dict(dk_in=torch.randn(1, CA, 3, device="cuda"))),
    (ValueError, lambda: dict(gen=binding.GenParams(torch.randn(9 * CA, CA + 1, device="cuda")))),
    (TypeError, lambda: dict(out=torch.empty(1, 6, 9, 8, device="cuda", dtype=torch.bfloat16))),
    (binding.EscError, lambda: dict(workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))),
])
def test_refuses(error, change):
    with pytest.raises(error):
        call(**change())


def backward(**change):
    a = dict(x=torch.randn(1, 6, 9, 8, device="cuda"), grad_out=torch.randn(1, 6, 9, 8, device="cuda"), Ca=CA,
             lk=torch.randn(CA, KS, KS, device="cuda"), workspace=binding.new_backward_workspace(1, CA, 9, 8, KS, 0))
    a.update(change)
    return binding.convattn_backward(**a)


def test_refuses_an_estimator_without_w_up():
    gen = binding.GenParams(None)
    with pytest.raises(binding.EscError):
        call(gen=gen)
    with pytest.raises(TypeError):
        backward(gen=gen)
    with pytest.raises(binding.EscError):   # nothing to allocate: the library sees the missing weight
        backward(gen=gen, grads={"grad_w_up": torch.zeros(9 * CA, CA, device="cuda")})


@pytest.mark.parametrize("number", [int, float, np.int64, np.float32, str])
def test_whole_numbers_of_any_type(number):
    # the integer arguments are what int() makes of them
    lk = torch.randn(CA * 11, device="cuda")
    x = torch.randn(1, 6, 9, 8, device="cuda")
    want = call(x=x, lk=torch.stack([lk[11 * c:11 * c + 9].view(KS, KS) for c in range(CA)]))
    assert torch.equal(call(x=x, Ca=number(CA), lk=lk, ks=number(KS), lk_channel_stride=number(11)), want)


@pytest.mark.parametrize("form", [dict, lambda d: list(d.items()), lambda d: tuple(d.items())])
def test_gradient_buffers_as_a_mapping_or_as_pairs(form):
    mine = {"grad_x": torch.empty(1, 6, 9, 8, device="cuda"), "grad_dk": None}
    given = form(mine)
    got = backward(grads=given)
    assert got["grad_x"] is mine["grad_x"] and set(got) == {"grad_x", "grad_lk", "grad_dk"}
    assert mine["grad_dk"] is None and given == form(mine)   # the caller's own is left as it was
    assert set(backward(grads=form({}))) == {"grad_x", "grad_lk", "grad_dk"}


def test_gradient_of_x_into_any_buffer_with_room():
    x, go, lk = torch.randn(1, 6, 9, 8, device="cuda"), torch.randn(1, 6, 9, 8, device="cuda"), torch.randn(CA, KS, KS, device="cuda")
    want = backward(x=x, grad_out=go, lk=lk)["grad_x"]
    for buf in (torch.empty(500, device="cuda"), torch.empty(2000, dtype=torch.uint8, device="cuda")):
        assert backward(x=x, grad_out=go, lk=lk, grads={"grad_x": buf})["grad_x"] is buf
        assert torch.equal(buf.view(torch.float32)[:432].view(1, 6, 9, 8), want)
    for small in (torch.empty(431, device="cuda"), torch.empty(1, 6, 9, 8, dtype=torch.bfloat16, device="cuda")):
        with pytest.raises(TypeError):
            backward(x=x, grad_out=go, lk=lk, grads={"grad_x": small})


def test_streams_and_given_outputs():
    x = torch.randn(1, 6, 9, 8, device="cuda")
    lk, ws, out = torch.randn(KS, KS, device="cuda"), binding.new_workspace(1, CA, 9, 8), torch.empty_like(x)
    want = binding.convattn_forward(x, CA, lk, ws)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    assert binding.convattn_forward(x, CA, lk, ws, out=out, stream=s) is out
    s.synchronize()
    assert torch.equal(out, want)


def test_the_current_stream_is_the_one_used():
    # no stream given: the call belongs behind what the current stream still has to do, here to fill x
    x, lk, ws = torch.zeros(1, 6, 9, 8, device="cuda"), torch.randn(KS, KS, device="cuda"), binding.new_workspace(1, CA, 9, 8)
    later, big = torch.randn(1, 6, 9, 8, device="cuda"), torch.randn(4096, 4096, device="cuda")
    want = binding.convattn_forward(later, CA, lk, ws)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        for _ in range(10):   # some milliseconds
            big = big @ big * 1e-4
        x.copy_(later)
        got = binding.convattn_forward(x, CA, lk, ws)
    s.synchronize()
    assert torch.equal(got, want)


@pytest.mark.parametrize("hidden", [0, 5])
def test_backward_writes_every_gradient_it_allocates(hidden):
    # the buffers are not cleared first: two calls with different junk in the allocator's memory agree
    x, go = torch.randn(2, 6, 9, 8, device="cuda"), torch.randn(2, 6, 9, 8, device="cuda")
    K = hidden or CA
    gen = binding.GenParams(torch.randn(9 * CA, K, device="cuda"), torch.randn(9 * CA, device="cuda"), hidden,
                            torch.randn(hidden, CA, device="cuda") if hidden else None,
                            torch.randn(hidden, device="cuda") if hidden else None)
    lk, ws = torch.randn(CA, KS, KS, device="cuda"), binding.new_backward_workspace(2, CA, 9, 8, KS, hidden)
    got = []
    for junk in (float("nan"), 7.0):
        pieces = [torch.full((n,), junk, device="cuda") for n in (2 * 6 * 72, 36 * K, 72, 36, 36, 20, 5)]
        del pieces
        got.append(binding.convattn_backward(x, go, CA, lk, ws, gen=gen))
        keep = {k: v.clone() for k, v in got[-1].items()}
        got[-1] = keep
    assert set(got[0]) == {"grad_x", "grad_lk", "grad_dk", "grad_w_up", "grad_b_up"} | ({"grad_w_down", "grad_b_down"} if hidden else set())
    assert all(torch.equal(got[0][k], got[1][k]) for k in got[0])
    acc = binding.convattn_backward(x, go, CA, lk, ws, gen=gen, accumulate=True,
                                    grads={k: v.clone() for k, v in got[0].items() if k != "grad_x"})
    for k in ("grad_lk", "grad_w_up", "grad_b_up"):
        torch.testing.assert_close(acc[k], 2 * got[0][k], rtol=1e-6, atol=0)

"""Bias gradients and losses of a training step, whose column sums are formed where the values are written: at the edges
of the rows that one workgroup sums (16 at a time in the loss kernel, up to eight times; 32 or 128 behind a product)."""
import numpy as np
import pytest
import torch

from paper_2302_13053_amd import harness as Hn

pytestmark = pytest.mark.gpu


def step64(X, y, W1, b1, Wc, bc):
    """Loss and bias gradients in 64 bits, and the sums of the magnitudes of the products the latter are made of."""
    act = (y >= 0)
    count = max(int(act.sum()), 1)
    pre = X.double() @ W1.double() + b1.double()
    A = pre.clamp(min=0) if Wc is not None else pre
    logits = A @ Wc.double() + bc.double() if Wc is not None else pre
    logp = torch.log_softmax(logits, 1)
    pick = y.clamp(min=0).long()[:, None]
    loss = -(logp.gather(1, pick)[:, 0] * act).sum() / count
    dL = torch.exp(logp)
    dL.scatter_add_(1, pick, torch.full_like(dL[:, :1], -1.0))
    dL *= act.double()[:, None] / count
    sums = [(dL.sum(0), dL.abs().sum(0))]
    if Wc is not None:
        on = (pre > 0).double()
        sums.append(((on * (dL @ Wc.double().T)).sum(0), (on * (dL.abs() @ Wc.double().abs().T)).sum(0)))
    return loss, sums


@pytest.mark.usefixtures("transform_family")
@pytest.mark.parametrize("n", [1, 15, 17, 31, 33, 127, 129, 4097, 32768 * 2 - 1, 32768 * 2 + 17, 32768 * 3 + 5, 300_001])
@pytest.mark.parametrize("h,c", [(33, 41), (256, 64), (300, 3), (0, 64), (40, 65)])
def test_bias_gradients_and_loss(n, h, c):
    g = torch.Generator(device="cuda").manual_seed(n + 1000 * h + c)
    rnd = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda").uniform_(-1.0, 1.0, generator=g)
    d_in = 12
    # products of 2^-7 and biases of odd multiples of 2^-8: the hidden sums are exact and never zero, so that no unit's
    # state hangs on a rounding
    X, W1 = (rnd(n, d_in) * 8).round() / 8, (rnd(d_in, h or c) * 16).round() / 16
    b1 = ((rnd(h or c) * 64).round() * 2 + 1) / 256
    Wc, bc = (rnd(h, c) / 8, rnd(c)) if h else (None, None)
    y = torch.randint(0, c, (n,), generator=g, device="cuda", dtype=torch.int32)
    if n > 1:
        y[torch.rand(n, generator=g, device="cuda") < 0.4] = -1
    loss, gW1, gb1, gWc, gbc = Hn.layer_grad(X, d_in, y, W1, b1, Wc, bc)
    want, sums = step64(X, y, W1, b1, Wc, bc)
    assert abs(float(loss[0]) - float(want)) <= 1e-5 * abs(float(want))
    for got, (total, size) in zip([gbc, gb1] if h else [gb1], sums):
        # every term is rounded like the products behind it (about 1e-6 of its size), and every float32 sum holds up to 32
        # terms in a row, then at most 50 partial sums in a row and a tree: below 100 roundings of 2^-24 of the terms
        err = (got.double() - total).abs()
        assert bool((err <= 1e-5 * size + 1e-30).all()), (n, h, c, float((err / (size + 1e-30)).max()))
    again = Hn.layer_grad(X, d_in, y, W1, b1, Wc, bc)
    for a, b in zip((loss, gW1, gb1, gWc, gbc), again):
        assert a is None or torch.equal(a, b)


@pytest.mark.parametrize("n,d_in,h,c", [(8000, 300, 256, 160), (5003, 131, 300, 131), (2708, 201, 500, 140)])
def test_products_in_halves(n, d_in, h, c):
    """Shapes of fewer than 128 blocks whose products are formed in halves of the sum, all three kinds: the forward, whose signs are
    decided, the product behind the ReLU's mask with its column sums, the input's gradient."""
    g = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda").uniform_(-1.0, 1.0, generator=g)
    X, W1 = (rnd(n, d_in) * 8).round() / 8, (rnd(d_in, h) * 16).round() / 16              # (exact hidden sums, as above)
    b1 = ((rnd(h) * 64).round() * 2 + 1) / 256
    Wc, bc = rnd(h, c) / 8, rnd(c)
    y = torch.randint(0, c, (n,), generator=g, device="cuda", dtype=torch.int32)
    y[torch.rand(n, generator=g, device="cuda") < 0.4] = -1
    gX = torch.empty(n, d_in, device="cuda")
    loss, gW1, gb1, gWc, gbc = Hn.layer_grad(X, d_in, y, W1, b1, Wc, bc, gX=gX)
    want, sums = step64(X, y, W1, b1, Wc, bc)
    assert abs(float(loss[0]) - float(want)) <= 1e-5 * abs(float(want))
    for got, (total, size) in zip([gbc, gb1], sums):
        assert bool(((got.double() - total).abs() <= 1e-5 * size + 1e-30).all())
    act = (y >= 0)
    pre = X.double() @ W1.double() + b1.double()
    dL = torch.softmax(pre.clamp(min=0) @ Wc.double() + bc.double(), 1)
    dL.scatter_add_(1, y.clamp(min=0).long()[:, None], torch.full_like(dL[:, :1], -1.0))
    dL *= act.double()[:, None] / int(act.sum())
    dA = (dL @ Wc.double().T) * (pre > 0)
    size = (dL.abs() @ Wc.double().abs().T) * (pre > 0)
    for got, total, terms in ((gX, dA @ W1.double().T, size @ W1.double().abs().T), (gW1, X.double().T @ dA, X.double().abs().T @ size)):
        assert bool(((got.double() - total).abs() <= 1e-5 * terms + 1e-30).all())

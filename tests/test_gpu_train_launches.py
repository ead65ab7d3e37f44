"""The training step's launches against each other: the optimiser inside the
reduction against the two entry points in turn, and the reduction over many
workgroups against the one of a single workgroup."""
import pytest
import torch

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

BOX = ((0.0, 0.0, 0.0), (8.0, 3.0, 8.0))


def _batch(gi, n, seed=7):
    g = torch.Generator("cuda").manual_seed(seed)
    b = gi.MlpBatch(max(n, 1))
    b.pos.copy_(torch.rand(max(n, 1), 4, device="cuda", generator=g) * 3.0)
    b.nrm.copy_(torch.nn.functional.normalize(torch.randn(max(n, 1), 4, device="cuda", generator=g), dim=1))
    b.target.copy_(torch.rand(max(n, 1), 4, device="cuda", generator=g) + 0.1)
    b.qprobe.copy_(torch.rand(max(n, 1), 4, device="cuda", generator=g))
    return b


# no workgroup, part of one, whole ones and one sample more; one group of the
# reduction's rows and one more; one round of groups and one more
@pytest.mark.parametrize("precision,ema", [("bf16", None), ("fp8", 0.95)])
@pytest.mark.parametrize("n", [0, 1, 64, 65, 1024, 1025, 16384, 16385])
def test_train_step_is_gradient_then_adam(n, precision, ema):
    from paper_2108_05263_amd import gi
    b = _batch(gi, n)
    b.target[::5, 3] = 0.0                 # invalid samples
    b.n = n
    ws, out = gi.train_workspace(n), []
    for fused in (True, False):
        m = gi.Mlp(*BOX, precision=precision, warmup_steps=2, ema_decay=ema)
        m.init(3)
        grad = torch.full((gi.MLP_N_PARAMS,), 7.0, device="cuda")
        for t in (1, 2):
            if fused:
                gi.mlp_train_step(m, b, t, 1e-2, ws)
            else:
                gi.mlp_grad(m, b, grad, ws)
                gi.mlp_adam(m, grad, t)
        torch.cuda.synchronize()
        assert m.state_words()["valid"] == n - (n + 4) // 5
        out.append([x.clone() for x in (m.params, m.adam_m, m.adam_v, m.weights, m.scales, m.state)] +
                   ([m.ema.clone()] if ema else []))
    for x, y in zip(*out):
        assert torch.equal(x.view(-1).view(torch.uint8), y.view(-1).view(torch.uint8))


@pytest.mark.parametrize("copies", [2, 16, 32, 256, 512])
def test_gradient_over_many_workgroups(copies):
    """A batch repeated 2^k times has the gradient of one copy: every partial
    is the same value over 2^k, so only the sums round, (16 + copies / 16) of
    them at 2^-24 each."""
    from paper_2108_05263_amd import gi
    m = gi.Mlp(*BOX)
    m.init(3)
    one = _batch(gi, 64)
    many = gi.MlpBatch(64 * copies)
    for k in ("pos", "nrm", "target", "qprobe"):
        getattr(many, k).copy_(getattr(one, k).repeat(copies, 1))
    grads = []
    for b in (one, many):
        grad = torch.zeros(gi.MLP_N_PARAMS, device="cuda")
        gi.mlp_grad(m, b, grad, gi.train_workspace(b.n))
        grads.append(grad.double())
    assert m.state_words()["valid"] == 64 * copies
    err = (grads[1] - grads[0]).abs() / grads[0].abs().clamp_min(1e-30)
    assert float(err.max()) <= (17 + copies / 16) * 2.0 ** -24

"""The cost model's kernels at the edges of their tiles (4 samples a training wave, 8 a forward one, 4 waves a
workgroup, at most 256 gradient parts, 64 inputs staged at a time), against the FP64 model."""
import numpy as np
import pytest

from oracle import mlp
from paper_0905_2203_amd import epi

pytestmark = pytest.mark.gpu


def relative(a, b):
    return float(np.linalg.norm(a.astype(np.float64) - b) / max(np.linalg.norm(b), 1e-30))


# A value is a sum of at most a few thousand FP32 products in chains of at most 256: an error of a few
# hundred roundings (2^-24 each) of terms no larger than the result's norm times a small factor.
TOLERANCE = 4096 * 2.0 ** -24


@pytest.mark.parametrize("F", [1, 24, 64, 65, 180])
@pytest.mark.parametrize("B", [1, 3, 4, 5, 8, 9, 33, 1023, 1024, 1025, 2100])
def test_forward_and_gradient(B, F):
    rng = np.random.default_rng(B * 1000 + F)
    X = rng.normal(size=(B, F)).astype(np.float32)
    t = rng.normal(size=B).astype(np.float32)
    p = rng.normal(scale=0.2, size=mlp.n_params(F)).astype(np.float32)
    with epi.Context(0) as ctx:
        ctx.epi_mlp_init(F, 1)
        ctx.epi_mlp_set_params(p)
        y = ctx.epi_mlp_forward(X)
        L, g = ctx.epi_mlp_grad(X, t)
    Lw, gw = mlp.grad(p.astype(np.float64), X, t.astype(np.float64))
    assert relative(y, mlp.forward(p.astype(np.float64), X)) < TOLERANCE
    assert abs(L - Lw) < TOLERANCE * max(1.0, Lw)
    assert relative(g, gw) < TOLERANCE


def test_training_steps_equal_gradient_and_adam():
    """An epoch of mini-batches (the last one shorter) is the gradient and the Adam step of each in turn."""
    rng = np.random.default_rng(4)
    B, F, batch = 1100, 24, 512
    X = rng.normal(size=(B, F)).astype(np.float32)
    t = rng.normal(size=B).astype(np.float32)
    p = rng.normal(scale=0.2, size=mlp.n_params(F)).astype(np.float32)
    with epi.Context(0) as ctx:
        ctx.epi_mlp_init(F, 1)
        ctx.epi_mlp_set_params(p)
        losses = ctx.epi_mlp_train(X, t, 2, batch, 3e-3)
        trained = ctx.epi_mlp_get_params()
        ctx.epi_mlp_set_params(p)
        want = []
        for _ in range(2):
            total = 0.0
            for b in range(0, B, batch):
                L, g = ctx.epi_mlp_grad(X[b:b + batch], t[b:b + batch])
                ctx.epi_mlp_adam_step(g, 3e-3)
                total += float(np.float32(L)) * len(t[b:b + batch])
            want.append(total / B)
        # (the same sums; the update may be contracted differently)
        assert relative(trained, ctx.epi_mlp_get_params().astype(np.float64)) < TOLERANCE
        assert relative(losses, np.array(want)) < TOLERANCE

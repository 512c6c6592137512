"""Screening-model convolutions at the edges of their tiles and load paths:
channel counts that are no multiple of 8 (element loads), images down to one
pixel at the deepest level, ragged pixel and output-channel tiles, and a batch
large enough for the 256-pixel tiles.

Predictions: against the CPU reference that rounds to bf16 where the GPU
stores it, to 5e-3 relative (L2) as in test_gpu_surrogate.py.

Gradients: the loss is a mean over labels and plans do not interact, so with
equal label counts and a power of two of plans the gradient of a batch is the
mean of its plans' gradients; scaling by a power of two is exact in bf16, so
the two sides take the same ReLU and pooling decisions on the same activations
and differ only in the float32 summation order over at most 1e6 pixels (2^-24
times a few hundred at worst on entries that cancel): 1e-4 relative (L2), and
on each layer.  The batch and the single plans run different tiles and
slices."""
import numpy as np
import pytest

from oracle import surrogate_ref as sr
from paper_2607_05818_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt,nx,ny,C,B", [(1, 8, 8, 4, 2), (4, 40, 24, 12, 4), (2, 24, 48, 20, 2),
                                          (3, 16, 72, 40, 2), (1, 128, 128, 4, 8)])
def test_shapes(nt, nx, ny, C, B):
    from paper_2607_05818_amd import reff
    print("[case] surrogate shapes", nt, nx, ny, C, B, flush=True)
    s = reff.reff_surrogate_create(nt, nx, ny, C, seed=3)
    p = reff.reff_surrogate_get_params(s)
    rng = np.random.default_rng([nt, nx, ny, C])
    p = np.where(sr.weight_mask(nt, C), p, rng.normal(scale=0.1, size=p.size)).astype(np.float32)
    reff.reff_surrogate_set_params(s, p)
    plans = [gen.small_random_desc(40 + i, nt, nx, ny, 12, 3) for i in range(B)]
    # labels on tiers without pads where there is one, so that every plan counts 16
    lo = nx * ny if nt > 1 else 0
    labels = []
    for d in plans:
        ids = np.setdiff1d(np.arange(lo, nt * nx * ny), gen.pad_ids(d))
        labels.append((rng.choice(ids, size=16, replace=False), rng.uniform(0.2, 3.0, 16)))
    pred = np.stack([np.log(np.where(r > 0, r, 1.0)) for r in reff.reff_surrogate_predict(s, plans)])
    _, _, rpred = sr.loss_and_grad(p, plans, labels, nt, nx, ny, C, emulate_bf16=True)
    free = np.ones((B, nt * nx * ny), dtype=bool)
    for b, d in enumerate(plans):
        free[b, gen.pad_ids(d)] = False
    rel = lambda a, b: np.linalg.norm(a - b) / np.linalg.norm(b)  # noqa: E731
    assert rel(pred[free], rpred.reshape(B, -1)[free]) <= 5e-3
    _, g = reff.reff_surrogate_loss_grad(s, plans, labels)
    one = [reff.reff_surrogate_loss_grad(s, [d], [v])[1].astype(np.float64) for d, v in zip(plans, labels)]
    mean = np.mean(one, axis=0)
    assert np.linalg.norm(mean) > 0
    assert rel(g, mean) <= 1e-4
    for name, (w, b) in sr.split(np.arange(p.size), nt, C).items():
        for part in (w, b):
            i = np.asarray(part.numpy(), dtype=np.int64).ravel()
            if np.linalg.norm(mean[i]) > 0:
                assert rel(g[i], mean[i]) <= 1e-4, name

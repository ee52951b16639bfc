"""GPU parity at the sizes where a tiled kernel can go wrong: edges of tiles, remainders, the
smallest and largest of a launch rule's range.  Against the float64 oracle, with the tolerances
of parity.py."""
import dataclasses

import pytest
import torch

import paper_2407_20485_amd as a2sf
from paper_2407_20485_amd import synth
import parity

pytestmark = pytest.mark.gpu


def variant(base, **kw):
    return dataclasses.replace(synth.CONFIGS[base], **kw)


def prompt_and_steps(w, alpha, sample=None, steps=2):
    """The prompt phase and a few steps in lock-step with the oracle, then the prompt phase without
    outputs: the same tokens, the scores to fp32 rounding."""
    p = parity.Problem(w, sample=sample)
    ls = parity.LockStep(p, alpha)
    ls.prefill()
    full = p.cache.snapshot()
    p.gpu_prefill(alpha, want_o=False, want_scores=False)
    torch.cuda.synchronize()
    assert torch.equal(full[3], p.cache.pos)
    assert torch.allclose(full[2], p.cache.scores, rtol=1e-5, atol=0.0)
    for t in range(steps):
        ls.step(t)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 97, 128, 129, 161, 300])
def test_fp32_prompt_tiles(n, d):
    """Tiles of 32 rows and keys, every fourth one to a wave: waves without a tile, ragged last
    tiles, one to ten tiles."""
    for alpha in (0.0, 0.7, 1.0):
        prompt_and_steps(variant(0, heads=3, d=d, n=n, T=2, select=min(9, n), recent=4, name="fp32 tiles"), alpha)

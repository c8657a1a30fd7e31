"""FDK pre-filter at the edges of its matrix-core tiles: row lengths around 16,
the chunks of 512 and the direct kernel's 2048, row counts around 16.  The sums
are FP64 on FP32-weighted pixels, so the bar is the existing 1e-5 of max|ref|."""
import math

import numpy as np
import pytest
import torch

from oracle import fdk as ofdk
from synth import Geom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu,nv,V", [(1, 1, 1), (2, 3, 1), (15, 16, 1), (16, 17, 1), (33, 5, 7),
                                     (128, 31, 1), (511, 3, 1), (512, 16, 2), (513, 2, 1), (1024, 2, 1),
                                     (1025, 3, 1), (2047, 1, 1), (2048, 2, 1), (2049, 1, 1)])
def test_rows(dp, nu, nv, V):
    g = Geom(8, 8, 8, 1.0, 1.0, 1.0, nu, nv, 0.4, 0.5, off_u=0.75, off_v=-0.25)
    x = np.random.default_rng(nu).standard_normal((V, nv, nu)).astype(np.float32)
    ref = ofdk.fdk_filter(g, x, math.pi / V)
    t = torch.tensor(x, device="cuda:0")
    got = dp.fdk_filter(g, t, math.pi / V)
    assert np.abs(got.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()
    dp.fdk_filter(g, t, math.pi / V, out=t)
    assert torch.equal(t, got)


def test_rows_do_not_mix(dp):
    g = Geom(8, 8, 8, 1.0, 1.0, 1.0, 70, 20, 0.4, 0.5)
    x = torch.randn((1, 20, 70), generator=torch.Generator().manual_seed(5)).cuda()
    want = dp.fdk_filter(g, x, 1.0)
    x[0, 7, 30] = math.inf
    got = dp.fdk_filter(g, x, 1.0)
    keep = torch.ones(20, dtype=torch.bool)
    keep[7] = False
    assert torch.equal(got[0, keep], want[0, keep])
    # the ramp's even taps are zero: inf reaches its own pixel and the odd distances
    odd = (torch.arange(70) - 30) % 2 == 1
    assert torch.isfinite(got[0, 7, ~odd.cuda()]).sum() == 34 and not torch.isfinite(got[0, 7, odd.cuda()]).any()


@pytest.mark.parametrize("nu,V", [(64, 95), (70, 95), (200, 20), (384, 12), (512, 12), (513, 11), (1025, 9), (2047, 8)])
def test_a_view_does_not_depend_on_its_launch(dp, nu, V):
    """Few rows take a kernel of their own: one view alone has the bits it has among
    many, in place too."""
    g = Geom(8, 8, 8, 1.0, 1.0, 1.0, nu, 90, 0.4, 0.5, off_u=0.75, off_v=-0.25)
    x = torch.randn((V, 90, nu), generator=torch.Generator().manual_seed(nu)).cuda()
    want = dp.fdk_filter(g, x, 0.1)
    for v in (0, V - 1):
        one = x[v:v + 1].clone()
        assert torch.equal(dp.fdk_filter(g, one, 0.1)[0], want[v])
        dp.fdk_filter(g, one, 0.1, out=one)
        assert torch.equal(one[0], want[v])

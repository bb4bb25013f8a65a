"""The drop threshold of the block orthonormalisation where it is not a finite number: a pivot is
kept when |R_jj|^2 > (tau ref)^2 (and only then), so an undefined threshold (0 times infinity) or
an infinite one keeps nothing, while a zero one keeps every direction of the block."""
import math

import numpy as np
import pytest
import torch

import paper_2308_01480_amd as ttr
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,s", [(40, 3), (961, 8), (300, 17), (960, 64)])
@pytest.mark.parametrize("ref,tau,keeps", [(math.inf, 0.0, False), (0.0, 1e200, False), (math.inf, 1e-10, False),
                                           (1.0, 1e200, False), (1.0, 0.0, True), (0.0, 0.0, True), (0.0, 1e-10, True)])
def test_undefined_threshold(m, s, ref, tau, keeps):
    announce(f"orth threshold m={m} s={s} ref={ref} tau={tau}")
    p = np.random.default_rng(m).standard_normal((m, s))
    q, k = ttr.orth(torch.from_numpy(p).cuda(), ref, tau)
    assert k == (s if keeps else 0)
    assert bool((q != 0).any()) == keeps

"""The exact Z at point counts around its tiles of 2048 points, its chunks of 32
and its rounds of 8, against the oracle's definition (1e-6, as the other tests of
it), with coincident points and with distances that overflow fp32 when squared."""
import pytest
import torch

import oracle
import paper_2212_11506_amd as bh
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 7, 9, 31, 33, 2047, 2048, 2049, 2055, 2081, 4095, 4097, 6145, 10_007])
@pytest.mark.parametrize("scale", [1.0, 1e25])
def test_z_exact_units(n, scale):
    Y = synth.random_y(n, n, scale=scale, dups=n // 3)
    Zo = oracle.z_exact(Y)
    Z = bh.z_exact(torch.from_numpy(Y).to("cuda:0"))
    # a pair's term is fp32: one below 2^-126 (points more than 1e19 apart) counts as 0
    assert abs(Z - Zo) <= 1e-6 * Zo + n * n * 2.0 ** -126

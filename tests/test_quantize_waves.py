"""Quantisation of long rows, eight and sixteen waves to a row: codes and scales against the oracle, bit for bit, with a last group, a last
k block and most lanes of the last pass missing, on both sides of the rule's lines."""
import numpy as np
import pytest

from paper_2409_17870_amd import binding, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("M, K", [(1, 8193), (9, 8704), (33, 11001), (2, 16384), (5, 16385), (257, 16400), (3, 32769), (1, 65537), (1030, 8200), (1030, 10752)])
def test_long_rows(M, K, p):
    import torch
    import oracle
    x = inputs.normal_features_f16(9100 + M + K + p, inputs.TAG_A, M, K, outlier_every=61)
    x[M - 1, K - 1] = 1000.0  # the largest magnitude is the very last element
    if M > 1:
        x[0, :] = 0
    want_codes, want_scale = oracle.quantize_rows(x, p)
    packed, scale = binding.apmm_quantize_pack_activations(torch.from_numpy(x).to("cuda:0"), p)
    assert np.array_equal(scale.cpu().numpy().view(np.uint16), want_scale)
    again = binding.apmm_pack_activations(torch.from_numpy(want_codes).to("cuda:0"), p)
    assert torch.equal(packed, again)

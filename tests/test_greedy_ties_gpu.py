"""Greedy verification of rows whose maximum is zero under both signs: -0.0 and
+0.0 are equal logits, so the lowest index is the argmax whichever vocabulary
segment (2 to 16 of them) holds which sign."""
import numpy as np
import pytest

from paper_2310_07177_amd import synth
from tests.test_parity_gpu import check_verify, osd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,dtype", [(8193, "bf16"), (32003, "bf16"), (65537, "bf16"), (131072, "bf16"),
                                     (8192, "f32"), (32768, "f32"), (65536, "f32")])
def test_zeros_of_both_signs(osd, V, dtype):
    B, K = 6, 2
    t = np.full((B, K + 1, V), -5.0, np.float32)
    g = np.random.default_rng(V)
    for b in range(B):
        for i in range(K + 1):  # the sign at the lowest id alternates
            ids = np.sort(g.choice(V, 4, replace=False))
            ids[0], ids[3] = 5 + i, V - 1 - b  # the first segment and the last
            t[b, i, ids] = np.float32([-0.0, 0.0, -0.0, 0.0]) * (1 if (b + i) % 2 == 0 else -1)
    tokens = np.full((B, K), 5, np.int32) + np.arange(K, dtype=np.int32)  # accepted: the lowest ids
    tokens[1, 1] = V - 2  # an equal logit at a higher id: rejected
    x = dict(target=synth.store(t, dtype), draft=None, tokens=tokens, u_accept=None, u_resample=None, T=0.0)
    check_verify(osd, x, f"zeros V={V} {dtype}", max_excluded_frac=0.0)

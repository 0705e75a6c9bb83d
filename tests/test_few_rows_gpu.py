"""Distillation of few rows of the longest streaming tile, which are split over
workgroups (up to one row per two CUs, V above 24576 bf16): both sides of either
limit, ragged and whole rows, with and without a mask, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2310_07177_amd import synth
from tests.test_parity_gpu import check_distill, osd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,V", [(1, 24576), (1, 24577), (3, 24584), (5, 32003), (2, 32768), (128, 24600),
                                    (129, 24600)])
@pytest.mark.parametrize("kind", ["fkl", "rkl", "jsd"])
def test_few_long_rows(osd, rows, V, kind):
    x = synth.verify_inputs(rows, 1, V, "bf16", T=1.0, seed=rows + V % 97, target_std=2.5, draft_noise=1.0)
    mask = (np.random.default_rng(rows).random((rows, 1)) < 0.6).astype(np.uint8)
    for m in (np.ones((rows, 1), np.uint8), mask):
        check_distill(osd, x["target"][:, :1].copy(), x["draft"], kind, 0.4, 1.2, m, f"rows={rows} V={V} {kind}")

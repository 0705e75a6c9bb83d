"""Distillation of few rows of the longest streaming tile, which are split over
workgroups (up to one row per two CUs, V above 24576 bf16): both sides of either
limit, ragged and whole rows, with and without a mask, against the fp64 oracle;
gradients written over the student rows; and where the one-call step and the
separate call give the same bits."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2310_07177_amd import synth
from tests._helpers import to_device
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


# (rows, V, dtype): a few rows of the longest tile, more, and shorter rows of either type.
IN_PLACE = [(3, 32000, "bf16"), (5, 24577, "bf16"), (200, 32768, "bf16"), (4, 8000, "bf16"), (4, 16383, "f32")]

CHILD = """
from tests import test_few_rows_gpu as t
import paper_2310_07177_amd as osd
for case in t.IN_PLACE:
    for kind in ("fkl", "rkl", "jsd"):
        t.check_in_place(osd, *case, kind)
print("IN_PLACE_OK", flush=True)
"""


def check_in_place(osd, rows, V, dtype, kind):
    import torch
    x = synth.verify_inputs(rows, 1, V, dtype, T=1.0, seed=rows, target_std=2.0, draft_noise=1.0)
    t = to_device(np.ascontiguousarray(x["target"][:, :1]))
    s = to_device(x["draft"])
    mask = torch.ones(rows, 1, dtype=torch.uint8, device=t.device)
    mask[1::3] = 0
    apart = s.clone()
    loss = torch.empty(2, dtype=torch.float32, device=t.device)
    div = torch.empty(rows, 1, dtype=torch.float32, device=t.device)
    osd.osd_distill_loss_grad(t, s, kind, 0.4, 1.0, mask=mask, out=(loss, div, s))
    want = osd.osd_distill_loss_grad(t, apart, kind, 0.4, 1.0, mask=mask)
    torch.cuda.synchronize()
    # Another kernel may take the call whose gradient lies elsewhere: last bits may differ.
    rtol = 2.0 ** -7 if dtype == "bf16" else 1e-4
    assert torch.allclose(s.float(), want[2].float(), rtol=rtol, atol=1e-6), (rows, V, kind)
    assert torch.allclose(div, want[1], rtol=1e-5, atol=1e-7) and torch.allclose(loss, want[0], rtol=1e-5, atol=1e-7)


def test_gradient_over_the_student_rows(osd):
    """With the bound on the split rows' waits set to 0 (in a child process: it is
    read once), a split row's segments are read again after siblings have written
    theirs; a gradient in the student rows' place takes the kernel that never does."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-u", "-c", CHILD], cwd=root, env=dict(os.environ, OSD_SPLIT_POLLS="0"),
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "IN_PLACE_OK" in r.stdout, r.stdout[-1000:] + r.stderr[-2000:]


@pytest.mark.parametrize("B,K,V,dtype", [(2, 3, 16000, "bf16"), (2, 3, 16000, "f32"), (2, 2, 40000, "bf16"),
                                         (64, 3, 32000, "bf16"), (2, 3, 32000, "bf16")])
@pytest.mark.parametrize("kind", ["fkl", "rkl", "jsd"])
def test_one_call_and_separate_call(osd, B, K, V, dtype, kind):
    import torch
    x = synth.verify_inputs(B, K, V, dtype, T=0.9, seed=7, target_std=2.0, draft_noise=1.0)
    t, s = to_device(x["target"]), to_device(x["draft"])
    one = osd.osd_verify_distill(t, s, to_device(x["tokens"]), to_device(x["u_accept"]), to_device(x["u_resample"]),
                                 0.9, kind, 0.4)
    two = osd.osd_distill_loss_grad(t, s, kind, 0.4, 0.9, B=B, K=K, teacher_batch_stride=(K + 1) * V,
                                    student_batch_stride=K * V)
    torch.cuda.synchronize()
    few = dtype == "bf16" and 24576 < V <= 32768 and B * K <= torch.cuda.get_device_properties(0).multi_processor_count // 2
    if few:  # another order of sums
        assert torch.allclose(one[4], two[1], rtol=1e-5, atol=1e-7)
        assert torch.allclose(one[5].float(), two[2].float(), rtol=2.0 ** -7, atol=1e-6)
    else:
        assert torch.equal(one[4], two[1]) and torch.equal(one[5], two[2])

"""Distillation of masked rows shared out among persistent workgroups: every row that
is on gets what it gets without a mask, every other zeros, and the loss is the sum
over the rows, with rows just above one per workgroup, several slices of flags, a
last slice of few rows, masks at odd addresses and masks of one kind only."""
import numpy as np
import pytest

from tests.test_fused_gpu import osd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

# (rows, V, dtype): 256 threads (slices of 4096 flags) and 1024 threads (slices of 16384).
CASES = [(257, 20000, "bf16"), (700, 17000, "f32"), (2049, 40, "bf16"), (4096, 2041, "bf16"), (4099, 8, "bf16"),
         (9001, 37, "f32"), (16385, 4100, "bf16"),
         # One row per CU and one more (the kernel for two workgroups on a CU); two rows per
         # workgroup and one more (the list), at one, two and seven workgroups on a CU.
         (256, 5000, "bf16"), (257, 5000, "bf16"), (512, 9000, "bf16"), (513, 9000, "bf16"), (1024, 8000, "f32"),
         (1025, 8000, "f32"), (3584, 600, "bf16"), (3585, 600, "f32")]


@pytest.mark.parametrize("rows,V,dtype", CASES)
@pytest.mark.parametrize("kind", ["fkl", "jsd"])
def test_masked_rows(osd, rows, V, dtype, kind):
    import torch
    g = torch.Generator(device="cuda").manual_seed(rows + V)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    t = (torch.randn(rows, 1, V, device="cuda", generator=g) * 2.5).to(td)
    s = (t.float() + torch.randn(rows, 1, V, device="cuda", generator=g)).to(td)
    _, every, grad = osd.osd_distill_loss_grad(t, s, kind, beta=0.3, tau=1.3)
    every, grad = every.clone(), grad.clone()
    store = torch.zeros(rows + 7, dtype=torch.uint8, device="cuda")
    for at, share in ((0, 0.4), (3, 0.9), (5, 0.0), (1, 1.0), (6, -1.0)):
        mask = store[at:at + rows].view(rows, 1)
        mask.copy_((torch.rand(rows, 1, device="cuda", generator=g) < share).to(torch.uint8) * 7)
        if share < 0:
            mask[rows - 1] = 1  # only the last row
        on = mask.bool()
        loss, row, out = osd.osd_distill_loss_grad(t, s, kind, beta=0.3, tau=1.3, mask=mask)
        assert torch.equal(row, torch.where(on, every, 0.0))
        assert torch.equal(out, torch.where(on.unsqueeze(-1), grad, torch.zeros_like(grad)))
        total, count = float(row.double().sum()), int(on.sum())
        # Each row's loss is rounded to fp32 (2^-24), and the sum once more.
        np.testing.assert_allclose(loss.double().cpu().numpy(), [total / max(count, 1), total], rtol=2.0 ** -22, atol=1e-30)

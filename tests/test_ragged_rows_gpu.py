"""Rows that are not 16-byte aligned, of lengths around every edge of the
kernels' tiles: a row shorter than one 16-byte chunk, exactly one, one element
more or less than a whole number of chunks or rounds, and whole rows that start
one element past an aligned address.  Every entry point is compared with the
fp64 oracle under the rules of the aligned rows (tests/_helpers.py).
"""
import numpy as np
import pytest

from oracle import ref
from paper_2310_07177_amd import synth
from tests._helpers import (MARGIN, compare_grad_bf16, compare_grad_f32, compare_losses, compare_verify, to_device)
from tests.test_fused_gpu import check_fused, osd  # noqa: F401  (the fixture)
from tests.test_shard_gpu import even_bounds, run_sharded
from tests.test_tree_gpu import check_tree

pytestmark = pytest.mark.gpu

# One chunk is 8 bf16 or 4 fp32 logits; the streaming tiles end at 2048, 4096,
# 8192, 16384, 24576 and 32768 bf16 logits (half as many fp32), the resident
# ones at 2048, 4096, 8192, 16384, 32768 and 65536.
STREAM = [("bf16", v) for v in (7, 8, 9, 2047, 2049, 4095, 8191, 8193, 16383, 16391, 24577, 32767)] + \
         [("f32", v) for v in (3, 4, 5, 1023, 1025, 4097, 12289, 16383)]
LONG = [("bf16", 32769), ("bf16", 50257), ("bf16", 65535), ("bf16", 65537), ("f32", 16385), ("f32", 32769)]


def shifted(a):
    """The array on the GPU, one element past an aligned address."""
    import torch
    t = to_device(a)
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    buf[1:] = t.reshape(-1)
    return buf[1:].view(t.shape)


@pytest.mark.parametrize("dtype,V", STREAM + LONG)
def test_verify_and_greedy(osd, dtype, V):
    import torch
    for T in (0.8, 0.0):
        x = synth.verify_inputs(5, 3, V, dtype, T=T, seed=V % 89, target_std=2.5, draft_noise=1.0, ragged=True)
        out = osd.osd_verify(to_device(x["target"]), None if T == 0 else to_device(x["draft"]),
                             to_device(x["tokens"]), None if T == 0 else to_device(x["u_accept"]),
                             None if T == 0 else to_device(x["u_resample"]), T, draft_len=to_device(x["draft_len"]))
        torch.cuda.synchronize()
        r = ref.verify(x["target"], None if T == 0 else x["draft"], x["tokens"], None if T == 0 else x["u_accept"],
                       None if T == 0 else x["u_resample"], T, draft_len=x["draft_len"])
        compare_verify(r, *[o.cpu().numpy() for o in out], f"V={V} {dtype} T={T}")


@pytest.mark.parametrize("dtype,V", [("bf16", v) for v in (8193, 16383, 16391, 32003, 32769, 50257, 65537)] +
                         [("f32", v) for v in (4097, 8191, 16383, 16385, 20001)])
def test_verify_many_rows(osd, dtype, V):
    """More rows than are split over workgroups (360: above one per CU), so the
    resident 512 x 4 and 512 x 8 tiles and the streaming kernel take them.  Most
    of the target's mass lies on the last tokens, so that draws end in the last
    chunk and the one it shares elements with; proposals of the last token ids are
    tested as well."""
    import torch
    B, K = 40, 8
    x = synth.verify_inputs(B, K, V, dtype, T=0.9, seed=V % 53, target_std=2.0, draft_noise=1.0, ragged=True)
    t = synth.as_f32(x["target"]).copy()
    t[1::2, :, V - 12:] += 11.0  # (every other sequence)
    x["target"] = synth.store(t, dtype)
    x["tokens"][2::4, 0] = V - 1
    x["tokens"][3::4, 0] = V - 1 - np.arange(B // 4) % 12
    assert x["target"].shape[0] * x["target"].shape[1] > torch.cuda.get_device_properties(0).multi_processor_count
    for u in (None, 0.0, 1.0 - 2.0 ** -24):  # as drawn; bonus draws; nearly every proposal rejected
        if u is not None:
            x["u_accept"] = np.full_like(x["u_accept"], u)
        out = osd.osd_verify(to_device(x["target"]), to_device(x["draft"]), to_device(x["tokens"]),
                             to_device(x["u_accept"]), to_device(x["u_resample"]), x["T"],
                             draft_len=to_device(x["draft_len"]))
        torch.cuda.synchronize()
        r = ref.verify(x["target"], x["draft"], x["tokens"], x["u_accept"], x["u_resample"], x["T"],
                       draft_len=x["draft_len"])
        n, _ = compare_verify(r, *[o.cpu().numpy() for o in out], f"V={V} {dtype} u={u}")
        assert n >= B * 3 // 4
        if u is not None:  # the draws did end in the last chunks
            extra = r["out_tokens"][np.arange(B), r["accepted_len"]][1::2]
            assert (extra >= V - 12).mean() > 0.5


@pytest.mark.parametrize("dtype,V", STREAM + [("bf16", 32769), ("f32", 16385)])
def test_fused_and_rejected(osd, dtype, V):
    import torch
    x = synth.verify_inputs(5, 3, V, dtype, T=0.9, seed=V % 83, target_std=2.0, draft_noise=1.0)
    mask = (np.random.default_rng(V).random((5, 3)) < 0.7).astype(np.uint8)
    for kind in ("jsd", "rkl"):
        check_fused(osd, x, kind, 0.4, mask, f"V={V} {dtype} {kind}")
    # The rejected rows only: the same decisions, and the distillation of reject_mask.
    out = osd.osd_verify_distill_rejected(to_device(x["target"]), to_device(x["draft"]), to_device(x["tokens"]),
                                          to_device(x["u_accept"]), to_device(x["u_resample"]), x["T"], "fkl")
    torch.cuda.synchronize()
    acc, toks, rmask = [o.cpu().numpy() for o in out[:3]]
    rv = ref.verify(x["target"], x["draft"], x["tokens"], x["u_accept"], x["u_resample"], x["T"])
    compare_verify(rv, acc, toks, rmask, f"V={V} {dtype} rejected")
    rd = ref.distill(x["target"], x["draft"], "fkl", beta=0.5, tau=x["T"], mask=rmask, B=5, K=3,
                     teacher_batch_stride=4 * V, student_batch_stride=3 * V)
    compare_losses(out[4].cpu().numpy(), rd["row_loss"], label=f"V={V} {dtype} rejected row loss")
    if dtype == "bf16":
        compare_grad_bf16(out[5].cpu().view(torch.int16).numpy().view(np.uint16), rd["grad"], f"V={V}")
    else:
        compare_grad_f32(out[5].cpu().numpy(), rd["grad"], f"V={V}")


@pytest.mark.parametrize("dtype,V", STREAM + LONG + [("bf16", 32000), ("f32", 8192)])
def test_distill_guarded(osd, dtype, V):
    """Loss and gradient from rows at odd addresses (aligned lengths among
    them); the gradient's neighbours in memory stay as they were."""
    import torch
    x = synth.verify_inputs(2, 2, V, dtype, T=1.0, seed=V % 79, target_std=2.0, draft_noise=1.0)
    t, s = x["target"][:, :2].copy(), x["draft"]
    mask = np.array([[1, 0], [1, 1]], np.uint8)
    td, sd = shifted(t), shifted(s)
    for kind in ("fkl", "jsd"):
        guard = torch.full((2 * 2 * V + 65,), 7.0, dtype=td.dtype, device=td.device)
        grad = guard[33:33 + 4 * V].view(2, 2, V)
        loss = torch.empty(2, dtype=torch.float32, device=td.device)
        rows = torch.empty(2, 2, dtype=torch.float32, device=td.device)
        osd.osd_distill_loss_grad(td, sd, kind, 0.5, 1.0, mask=to_device(mask), out=(loss, rows, grad))
        torch.cuda.synchronize()
        assert bool((guard[:33] == 7).all()) and bool((guard[33 + 4 * V:] == 7).all())
        rd = ref.distill(t, s, kind, beta=0.5, tau=1.0, mask=mask, B=2, K=2, teacher_batch_stride=2 * V,
                         student_batch_stride=2 * V)
        compare_losses(rows.cpu().numpy(), rd["row_loss"], label=f"V={V} {dtype} {kind}")
        if dtype == "bf16":
            compare_grad_bf16(grad.cpu().view(torch.int16).numpy().view(np.uint16), rd["grad"], f"V={V} {kind}")
        else:
            compare_grad_f32(grad.cpu().numpy(), rd["grad"], f"V={V} {kind}")


@pytest.mark.parametrize("dtype,V", STREAM)
def test_tree(osd, dtype, V):
    g = synth.rng(V)
    for T in (1.0, 0.0):
        x = synth.tree_inputs(3, np.stack([synth.random_tree_parents(g, 9) for _ in range(3)]), V, dtype, T=T,
                              seed=V % 73, target_std=2.0, draft_noise=1.0)
        check_tree(osd, x, f"V={V} {dtype} T={T}", max_excluded_frac=0.34)


@pytest.mark.parametrize("dtype,V", STREAM + LONG)
@pytest.mark.parametrize("N", [3, 600])
def test_sample(osd, dtype, V, N):
    """A few rows (split over workgroups) and more than two per CU, whose row
    stride is odd as well: one row, a mixture and the argmax."""
    import torch
    if N == 600 and V > 33000:
        N = 520
    x = synth.sample_inputs(N, V + 1, dtype, seed=V % 71, p_std=2.0)
    pd, qd = to_device(x["p"])[:, 1:], to_device(x["q"])[:, 1:]
    p, q = x["p"][:, 1:], x["q"][:, 1:]
    some = slice(None) if N < 10 else slice(N - 4, N)  # the oracle checks a few rows of many
    for T, beta in ((0.9, 0.0), (0.9, 0.3), (0.0, 0.0)):
        got = osd.osd_sample(pd, qd, T, beta, None if T == 0 else to_device(x["u"]))
        torch.cuda.synchronize()
        r = ref.sample(p[some].copy(), q[some].copy(), T, beta, None if T == 0 else x["u"][some])
        bad = (got.cpu().numpy()[some] != r["tokens"]) & ~(np.nan_to_num(r["margin"], nan=np.inf) < MARGIN)
        assert not bad.any(), (V, dtype, N, T, beta, np.nonzero(bad)[0])


@pytest.mark.parametrize("dtype,V,G", [("bf16", 21, 3), ("bf16", 8191, 2), ("bf16", 32003, 4), ("f32", 12289, 3)])
def test_shard(osd, dtype, V, G):
    for T in (0.8, 0.0):
        x = synth.verify_inputs(5, 3, V, dtype, T=T, seed=V % 67, target_std=2.5, draft_noise=1.0, ragged=True)
        acc, toks, rmask = run_sharded(osd, x, even_bounds(V, G))[:3]
        r = ref.verify(x["target"], None if T == 0 else x["draft"], x["tokens"], None if T == 0 else x["u_accept"],
                       None if T == 0 else x["u_resample"], T, draft_len=x["draft_len"])
        compare_verify(r, acc, toks, rmask, f"shard V={V} {dtype} T={T}")

"""Verification of rows split over workgroups (long rows, and few rows) against
the oracle: every segment count and tile, forced draws of both kinds, rows whose
draw falls back to p, and the bounded wait's fallback."""
import os
import subprocess
import sys

import numpy as np
import pytest

from oracle import ref
from paper_2310_07177_amd import synth
from tests._helpers import compare_verify, to_device
from tests.test_fused_gpu import osd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

# (B, K, V, dtype): 256 x 1, 256 x 2, 256 x 4 and 512 x 4 chunks per segment, 3 to 8 segments.
CASES = [(2, 4, 4104, "bf16"), (3, 3, 9001, "bf16"), (1, 4, 32000, "bf16"), (8, 5, 32003, "bf16"),
         (40, 3, 40000, "bf16"), (5, 8, 65535, "bf16"), (3, 2, 65537, "bf16"), (2, 2, 131072, "bf16"),
         (2, 4, 2052, "f32"), (4, 4, 8191, "f32"), (30, 2, 20001, "f32"), (2, 3, 65536, "f32"),
         # Both sides of the limits on few rows (256 CUs): 64 and 65 fp32 rows, 32 and 33 bf16 ones.
         (3, 4, 8193, "f32"), (16, 3, 16001, "f32"), (13, 4, 16384, "f32"), (8, 3, 16384, "bf16"), (11, 2, 16383, "bf16")]


def inputs(B, K, V, dtype):
    return synth.verify_inputs(B, K, V, dtype, T=0.9, seed=(B * 31 + V) % 97, target_std=2.5, draft_noise=1.0,
                               ragged=True)


def run(osd, x):
    import torch
    out = osd.osd_verify(to_device(x["target"]), to_device(x["draft"]), to_device(x["tokens"]),
                         to_device(x["u_accept"]), to_device(x["u_resample"]), x["T"],
                         draft_len=to_device(x.get("draft_len")))
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in out]


def oracle(x):
    return ref.verify(x["target"], x["draft"], x["tokens"], x["u_accept"], x["u_resample"], x["T"],
                      draft_len=x.get("draft_len"))


@pytest.mark.parametrize("B,K,V,dtype", CASES)
def test_split_rows(osd, B, K, V, dtype):
    x = inputs(B, K, V, dtype)
    for u in (None, 0.0, 1.0 - 2.0 ** -24):  # as drawn; every proposal accepted; nearly every one rejected
        if u is not None:
            x["u_accept"] = np.full_like(x["u_accept"], u)
        for _ in range(3):  # the workspace is left zero
            compare_verify(oracle(x), *run(osd, x), f"B={B} V={V} {dtype} u={u}")


@pytest.mark.parametrize("V,dtype", [(4104, "bf16"), (32000, "bf16"), (70001, "bf16"), (30000, "f32")])
def test_split_edges(osd, V, dtype):
    """Points at the ends of the CDF, identical rows (a forced rejection has no
    residual mass: the token comes from p), rows without a finite or with a NaN
    logit, proposals outside the vocabulary and invalid lengths."""
    x = synth.verify_inputs(6, 3, V, dtype, T=1.0, seed=5, target_std=2.0, draft_noise=1.0)
    for u in (0.0, 1.0 - 2.0 ** -24):
        x["u_resample"] = np.full_like(x["u_resample"], u)
        compare_verify(oracle(x), *run(osd, x), f"V={V} u_res={u}")
    same = dict(x, draft=x["target"][:, :3].copy(), u_accept=np.ones_like(x["u_accept"]))
    acc, toks, _ = run(osd, same)  # u = 1 rejects although p = q
    assert (acc == 0).all() and ((toks[:, 0] >= 0) & (toks[:, 0] < V)).all()
    inf, nan = (0xFF80, 0x7FC0) if dtype == "bf16" else (-np.inf, np.nan)
    bad = dict(x, target=x["target"].copy(), tokens=x["tokens"].copy(), draft_len=np.array([3, 0, 4, 3, 2, 3], np.int32))
    bad["target"][0, 0, :] = inf
    bad["target"][3, 0, V - 1] = nan
    bad["tokens"][5, 2] = V
    acc, toks, rmask = run(osd, bad)
    assert acc[[0, 1, 2, 3, 5]].tolist() == [-1] * 5 and (toks[[0, 1, 2, 3, 5]] == -1).all()
    r = oracle(dict(x, draft_len=np.full(6, 2, np.int32)))
    assert acc[4] == r["accepted_len"][4] and (toks[4] == r["out_tokens"][4]).all()


FALLBACK = """
import sys, numpy as np
import paper_2310_07177_amd as osd
from tests import test_verify_split_gpu as t
out = {}
for k, c in enumerate(t.CASES):
    for j, o in enumerate(t.run(osd, t.inputs(*c))):
        out[f"{k}_{j}"] = o
np.savez(sys.argv[1], **out)
print("FALLBACK_OK", flush=True)
"""


def test_split_fallback(osd, tmp_path):
    """With the bound on the waits set to 0 (read once per process, so in a
    child process) every segment computes its row's records itself; the
    results are those of the exchanging path."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    path = str(tmp_path / "fallback.npz")
    r = subprocess.run([sys.executable, "-u", "-c", FALLBACK, path], cwd=root, env=dict(os.environ, OSD_VERIFY_POLLS="0"),
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "FALLBACK_OK" in r.stdout, r.stderr[-2000:]
    got = np.load(path)
    for k, c in enumerate(CASES):
        for j, o in enumerate(run(osd, inputs(*c))):
            assert np.array_equal(o, got[f"{k}_{j}"]), (c, j)

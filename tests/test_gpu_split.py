"""GPU parity of the split-K forward (Sec. 3.3) against the fp64 oracle, and
agreement with the single-pass forward, on shapes with few query rows per head
(the regime the split targets) and on ragged, causal and empty-chunk cases."""
import numpy as np
import pytest

import oracle
from paper_2606_20005_amd import inputs
from parity_utils import KL_ATOL, KL_RTOL, check_rows, upload

pytestmark = pytest.mark.gpu


def run_split(sk, d, causal, direction, splits, workspace=None):
    import torch
    w = d["w"]
    q1, k1, q2, k2 = upload(d)
    out = sk.fwd_split(q1, k1, q2, k2, w.s1, w.s2, causal, direction, splits=splits, workspace=workspace)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out], (q1, k1, q2, k2)


@pytest.mark.parametrize("nq,nk,causal,direction,splits", [
    (1, 4000, False, 0, 7),       # one query row, ragged key tail
    (16, 4096, False, 0, 32),     # decode-like
    (16, 4096, True, 1, 5),       # causal bottom-right, reverse direction
    (33, 1000, True, 0, 3),       # two waves' worth of rows
    (200, 300, True, 0, 4),       # several query workgroups; the single pass of this shape takes the key split
    (64, 40, False, 0, 8),        # more splits than key tiles: empty chunks
    (300, 100, True, 0, 2),       # rows with no visible key (N_Q > N_K)
])
def test_split_matches_oracle(gpu_lib, nq, nk, causal, direction, splits):
    d = inputs.make("tiny", B=2, H=2, n_q=nq, n_k=nk)
    w = d["w"]
    (kl, l1, l2), _ = run_split(gpu_lib, d, causal, direction, splits)
    ref = oracle.forward(d["Q1"], d["K1"], d["Q2"], d["K2"], w.s1, w.s2, causal, direction)
    check_rows("kl", kl, ref[0])
    check_rows("lse1", l1, ref[1])
    check_rows("lse2", l2, ref[2])


@pytest.mark.parametrize("d1,d2", [(128, 128), (192, 64), (64, 256)])
def test_split_agrees_with_single_pass(gpu_lib, d1, d2):
    import torch
    d = inputs.make("tiny", B=1, H=4, n_q=48, n_k=3000, d1=d1, d2=d2, s1=d1 ** -0.5, s2=d2 ** -0.5)
    w = d["w"]
    (kl, l1, l2), (q1, k1, q2, k2) = run_split(gpu_lib, d, True, 0, "auto")
    one = [t.cpu().numpy() for t in gpu_lib.fwd(q1, k1, q2, k2, w.s1, w.s2, True, 0)]
    torch.cuda.synchronize()
    assert gpu_lib.split_count(1, 4, 48, 3000, d1, d2) > 1
    for got, ref in zip((kl, l1, l2), one):
        # the merge reorders fp32 sums: same value up to rounding
        assert np.allclose(got, ref, rtol=2e-5, atol=2e-5), float(np.max(np.abs(got - ref)))


def test_split_ignores_workspace_contents(gpu_lib):
    import torch
    d = inputs.make("tiny", B=1, H=2, n_q=20, n_k=2000)
    w = d["w"]
    ws = torch.full((gpu_lib.split_workspace_bytes(1, 2, 20, 6) // 4,), float("nan"), dtype=torch.float32,
                    device="cuda")
    (kl, _, _), _ = run_split(gpu_lib, d, False, 0, 6, workspace=ws)
    ref = oracle.forward(d["Q1"], d["K1"], d["Q2"], d["K2"], w.s1, w.s2, False, 0)
    check_rows("kl", kl, ref[0])


def test_split_one_is_the_single_pass(gpu_lib):
    import torch
    d = inputs.make("tiny", B=1, H=2, n_q=100, n_k=500)
    w = d["w"]
    (kl, l1, l2), (q1, k1, q2, k2) = run_split(gpu_lib, d, True, 0, 1)
    one = [t.cpu().numpy() for t in gpu_lib.fwd(q1, k1, q2, k2, w.s1, w.s2, True, 0)]
    torch.cuda.synchronize()
    for got, ref in zip((kl, l1, l2), one):
        assert np.array_equal(got, ref)


def test_autograd_uses_split_for_few_rows(gpu_lib):
    """attention_kl picks the adaptive split count; its values and gradients
    match the oracle on a decode-like shape."""
    import torch
    d = inputs.make("tiny", B=2, H=2, n_q=8, n_k=2048)
    w = d["w"]
    q1, k1, q2, k2 = (t.clone().requires_grad_(True) for t in upload(d))
    assert gpu_lib.split_count(2, 2, 8, 2048, 64, 64) > 1
    kl = gpu_lib.attention_kl(q1, k1, q2, k2, s1=w.s1, s2=w.s2)
    kl.sum().backward()
    torch.cuda.synchronize()
    ref = oracle.backward(d["Q1"], d["K1"], d["Q2"], d["K2"], w.s1, w.s2, False, 0)
    check_rows("kl", kl.detach().cpu().numpy(), ref[0])
    for name, got, r in (("dq2", q2.grad, ref[5]), ("dk2", k2.grad, ref[6])):
        g = got.float().cpu().numpy()
        assert np.linalg.norm(g - r) <= 1e-2 * np.linalg.norm(r), name


@pytest.mark.parametrize("splits", [2, 3, 16, 17, 33, 64, 65, 130])
@pytest.mark.parametrize("n_q", [1, 7, 65])
def test_merge_lanes_follow_the_split_count(gpu_lib, splits, n_q):
    """The merge gives a row 2, 4, ..., 64 lanes (powers of two around every edge, more partials than lanes) and a wave
    64 down to 1 rows, the last wave partly filled: every row against the single pass, which merges nothing."""
    import torch
    d = inputs.make("tiny", B=1, H=3, n_q=n_q, n_k=4200)
    w = d["w"]
    got, (q1, k1, q2, k2) = run_split(gpu_lib, d, False, 0, splits)
    one = [t.cpu().numpy() for t in gpu_lib.fwd(q1, k1, q2, k2, w.s1, w.s2, False, 0)]
    torch.cuda.synchronize()
    for a, b in zip(got, one):   # the merge reorders fp32 sums: same value up to rounding
        assert np.allclose(a, b, rtol=2e-5, atol=2e-5), float(np.max(np.abs(a - b)))

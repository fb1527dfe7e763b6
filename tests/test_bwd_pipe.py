"""The pipelined backward kernels: they compile without spilling, and they give the gradients of the plain kernels bit for
bit. A head's gradients do not depend on how many heads a call holds, while the kernel that computes them does: few
workgroups take the pipelined form with one row block per wave, more take the plain one, and many that stream enough rows
the pipelined form with two. That each call below takes the form it is meant to is asked of the host's rule itself."""
import concurrent.futures as cf
import os
import re
import subprocess

import numpy as np
import pytest

import oracle
from paper_2606_20005_amd import build, inputs
from parity_utils import check_grad, to_gpu_f32, upload

ALL = ("dq1", "dk1", "dq2", "dk2")
STUDENT, TEACHER = ("dq2", "dk2"), ("dq1", "dk1")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """The host's rule itself: rule(kernel, want, d1, d2, heads, nq, nk, causal) is 0 for the plain kernel of a call
    without reversed direction, else the pipelined kernel's row blocks per wave."""
    exe = str(tmp_path_factory.mktemp("rule") / "pipe_rule")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "pipe_rule.hip")
    r = subprocess.run([build.hipcc(), *build.CFLAGS, "--offload-host-only", src, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def ask(kernel, want, d1, d2, heads, nq, nk, causal, s1=0.125, s2=0.125):
        mode = (1 if "dq2" in want else 0) | (2 if "dq1" in want else 0)
        line = f"{int(kernel == 'dk')} {mode} {d1} {d2} {heads} {nq} {nk} {int(causal)} {s1:.9g} {s2:.9g}\n"
        return int(subprocess.run([exe], input=line, capture_output=True, text=True, check=True).stdout)
    return ask


def test_no_spills(tmp_path):
    """Every instantiation, at the flags of the build."""
    units = [f"kl_bwd_pipe_{k}_m{m}" for k in ("dq", "dk") for m in (1, 2, 3)]

    def remarks(u):
        src = f"{build.CSRC}/{u}.hip"
        r = subprocess.run([build.hipcc(), *build.CFLAGS, *build.unit_flags(src), "--offload-device-only", "-c", src, "-o",
                            str(tmp_path / f"{u}.o"), "-Rpass-analysis=kernel-resource-usage"], capture_output=True,
                           text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return r.stderr

    seen = 0
    with cf.ThreadPoolExecutor(len(units)) as ex:
        for text in ex.map(remarks, units):
            for name, spill in re.findall(r"Function Name: (\S*pipe_kernel\S*).*?ScratchSize \[bytes/lane\]: (\d+)", text,
                                          re.S):
                seen += 1
                assert spill == "0", name
    # modes 1 and 2: 16 pairs with one block, 5 with two; mode 3: 10 pairs for dQ, 6 for dK; causal and not
    assert seen == 2 * (2 * 2 * (16 + 5) + 10 + 6)


# heads, nq, nk, causal; heads of the part of them that takes the plain kernels and of the part that takes one block; the
# kernels for which this holds, and of which the whole call takes two blocks where they exist (under the mask for the
# gradients of the narrower head)
GRIDS = [
    (512, 70, 16400, False, 300, 30, ("dq",)), (512, 1, 16385, False, 300, 30, ("dq",)),
    (520, 4101, 70, False, 300, 30, ("dk",)), (130, 4200, 16500, False, 7, 1, ("dk",)),
    (8, 8100, 66000, True, 5, 2, ("dq",)), (32, 17000, 16700, True, 5, 3, ("dq", "dk")),
    (32, 16400, 16400, True, 4, 3, ("dq", "dk")),
]
DIMS = [(128, 128, STUDENT), (128, 64, STUDENT), (64, 128, STUDENT), (192, 64, STUDENT), (256, 64, STUDENT), (128, 64, TEACHER),
        (64, 192, TEACHER), (64, 64, STUDENT), (64, 64, ALL)]


@pytest.mark.parametrize("heads,nq,nk,causal,plain,one,kernels", GRIDS)
def test_grids_take_the_forms_they_compare(rule, heads, nq, nk, causal, plain, one, kernels):
    for d1, d2, want in DIMS:
        own, other = (d2, d1) if want == STUDENT else (d1, d2)
        two = want != ALL and own + other >= 192 and (not causal or own < other)
        for k in kernels:
            assert rule(k, want, d1, d2, heads, nq, nk, causal) == (2 if two else 0), (k, d1, d2, want)
            assert rule(k, want, d1, d2, plain, nq, nk, causal) == 0, (k, d1, d2, want)
            assert rule(k, want, d1, d2, one, nq, nk, causal) == 1, (k, d1, d2, want)


@pytest.mark.gpu
@pytest.mark.parametrize("heads,nq,nk,causal,plain,one,kernels", GRIDS)
@pytest.mark.parametrize("d1,d2,want", DIMS)
def test_same_bits_at_every_grid_size(gpu_lib, heads, nq, nk, causal, plain, one, kernels, d1, d2, want):
    """Ragged tiles, one-row tiles, rows without keys, negative and zero upstream gradients."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(nq * 1000 + nk)

    def normal(n, d):
        return torch.randn(1, heads, n, d, generator=gen, device="cuda").to(torch.bfloat16)

    t = [normal(nq, d1), normal(nk, d1), normal(nq, d2), normal(nk, d2)]
    g = torch.rand(1, heads, nq, generator=gen, device="cuda") + 0.5
    g[:, 1::3, ::5] *= -1.0   # every third head has negative values
    g[..., 3::7] = 0.0
    stats = gpu_lib.fwd(*t, causal=causal)

    def grads(lo, hi):
        u = [x[:, lo:hi].contiguous() for x in (*t, *stats, g)]
        out = gpu_lib.bwd(*u, causal=causal, want=want)
        return [x for x in out if x is not None]

    whole = grads(0, heads)
    for lo, hi in ((0, plain), (heads - one, heads)):
        for a, b in zip(whole, grads(lo, hi)):
            assert torch.isfinite(b).all()
            assert torch.equal(a[:, lo:hi], b), (lo, hi)


@pytest.mark.gpu
@pytest.mark.parametrize("d1,d2,want", [(256, 64, ("dq2", "dk2")), (192, 128, ("dq2", "dk2")), (256, 256, ("dq1", "dk1")),
                                        (128, 128, ALL), (64, 192, ALL), (64, 256, ("dq1", "dk1"))])
@pytest.mark.parametrize("nq,nk,causal", [(130, 200, True), (40, 33, False), (530, 600, True), (260, 33, False)])
def test_wide_heads_key_gradients_match_the_plain_kernel(gpu_lib, d1, d2, want, nq, nk, causal):
    """Wide heads take the pipelined kernels from 128 or 256 streamed rows on (the last two sizes); dK without a dQ in the
    call takes the plain kernel, which forms the row statistics itself."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(d1 * 7 + d2)
    t = [torch.randn(2, 3, n, d, generator=gen, device="cuda").to(torch.bfloat16)
         for n, d in ((nq, d1), (nk, d1), (nq, d2), (nk, d2))]
    g = torch.randn(2, 3, nq, generator=gen, device="cuda")
    stats = gpu_lib.fwd(*t, causal=causal)
    both = gpu_lib.bwd(*t, *stats, g, causal=causal, want=want)
    alone = gpu_lib.bwd(*t, *stats, g, causal=causal, want=[n for n in want if n.startswith("dk")])
    for n, a, b in zip(ALL, both, alone):
        if n.startswith("dk") and n in want:
            assert torch.equal(a, b), n


EXTREME_SCALES = [   # s1, s2 and the factor on Q and K that keeps the logits of order one
    (2.0 ** -98, 2.0 ** -102, 2.0 ** 45), (2.0 ** 30, 2.0 ** 29, 2.0 ** -16)]


def test_extreme_scales_take_the_plain_kernels(rule):
    for kernel in ("dq", "dk"):
        assert rule(kernel, ("dq2", "dk2"), 64, 64, 2, 600, 600, True) == 1
        for s1, s2, _ in EXTREME_SCALES:
            assert rule(kernel, ("dq2", "dk2"), 64, 64, 2, 600, 600, True, s1=s1) == 0
            assert rule(kernel, ("dq2", "dk2"), 64, 64, 2, 600, 600, True, s2=s2) == 0


@pytest.mark.parametrize("d1,d2", [(128, 64), (192, 64), (64, 128), (128, 128)])
@pytest.mark.parametrize("heads,nq,nk", [(1024, 8300, 290), (256, 8192, 1024), (64, 20000, 4000)])
def test_causal_rows_without_a_key_are_not_streamed(rule, heads, nq, nk, d1, d2):
    """A key of a causal head with nk < nq streams nk / 2 rows on average, however many rows there are."""
    assert rule("dk", STUDENT, d1, d2, heads, nq, nk, True) == 0
    assert rule("dk", STUDENT, d1, d2, heads, nq, nk, False) == 2


@pytest.mark.parametrize("d1,d2,alone", [(128, 128, False), (64, 64, False), (256, 256, True), (128, 192, True)])
def test_short_streams_take_the_plain_kernels(rule, d1, d2, alone):
    """One block starts to pay from 256 streamed rows for dK and 128 for dQ; where the plain kernel has one wave per SIMD,
    from 128 and at once."""
    for n, dq, dk in ((1000, 1, 1), (256, 1, 1), (255, 1, int(alone)), (128, 1, int(alone)), (127, int(alone), 0),
                      (1, int(alone), 0)):
        assert rule("dq", STUDENT, d1, d2, 8, 300, n, False) == dq, n
        assert rule("dk", STUDENT, d1, d2, 8, n, 300, False) == dk, n
    # rows without a key do not count for dQ
    assert rule("dq", STUDENT, d1, d2, 1, 30000, 600, True) == rule("dk", STUDENT, d1, d2, 1, 30000, 600, True) == 1
    assert rule("dq", STUDENT, d1, d2, 1, 30000, 500, True) == int(alone)


def test_causal_grids_over_one_round(rule):
    """Two workgroups to a CU: one after the other pays where their lengths differ enough (square heads), not where the
    blocks are of nearly one length (the last rows of a long context)."""
    for kernel in ("dq", "dk"):
        for heads, n in ((16, 4096), (8, 8192), (12, 4096), (4, 16384)):
            assert rule(kernel, STUDENT, 128, 128, heads, n, n, True) == 1, (kernel, heads, n)
            assert rule(kernel, STUDENT, 128, 128, heads, n, n, False) != 1, (kernel, heads, n)
        for heads, n in ((256, 256), (128, 512), (62, 979), (49, 1204)):   # the second start is not paid back
            assert rule(kernel, STUDENT, 128, 128, heads, n, n, True) == 0, (kernel, heads, n)
        assert rule(kernel, STUDENT, 128, 128, 8, 4096, 4096, True) == 1
    for heads, nq, nk in ((12, 5000, 60000), (8, 8192, 131072), (32, 2048, 36096)):
        assert rule("dq", STUDENT, 64, 128, heads, nq, nk, True) == 0
    for heads, nq, nk in ((7, 400, 8000), (16, 600, 4096)):
        assert rule("dk", STUDENT, 128, 128, heads, nq, nk, True) == 0


def test_two_blocks_where_they_were_measured(rule):
    """Under the mask only for the gradients of the narrower head and over four rounds: square heads from 16384 rows on,
    with a head dim four times as wide from 8192 (dK) and 12288 (dQ) on; without a mask also at equal dims, dQ on grids
    that fill their rounds."""
    for kernel, least in (("dk", 8192), ("dq", 12288)):
        for want, d1, d2 in ((STUDENT, 128, 64), (STUDENT, 192, 64), (STUDENT, 256, 64), (TEACHER, 64, 128), (TEACHER, 64, 256)):
            n = least if 256 in (d1, d2) else 16384
            assert rule(kernel, want, d1, d2, 32, 65536, 65536, True) == 2
            assert rule(kernel, want, d1, d2, 32, n, n, True) == 2
            assert rule(kernel, want, d1, d2, 32, n - 10, n - 10, True) == 0
            assert rule(kernel, want, d1, d2, 15, 16384, 16384, True) == 0   # 960 workgroups
        for want, d1, d2 in ((STUDENT, 128, 128), (TEACHER, 128, 128), (STUDENT, 64, 128), (TEACHER, 128, 64)):
            assert rule(kernel, want, d1, d2, 32, 65536, 65536, True) == 0
            assert rule(kernel, want, d1, d2, 32, 16384, 16384, False) == 2
    for causal in (False, True):   # rounds of equally long blocks: full ones, under the mask together with dK
        assert rule("dq", STUDENT, 192, 64, 8, 8192, 131072, causal) == 2
        assert rule("dq", STUDENT, 192, 64, 8, 7424, 131072, causal) == rule("dq", STUDENT, 192, 64, 9, 8192, 131072, causal) == 0
        assert rule("dq", STUDENT, 192, 64, 32, 2048, 60000, causal) == (0 if causal else 2)
        assert rule("dq", STUDENT, 192, 64, 16, 8192, 60000, causal) == (0 if causal else 2)
    assert rule("dq", STUDENT, 128, 128, 8, 8192, 131072, True) == 0
    for heads, nq, nk in ((64, 4385, 14421), (32, 40000, 7000)):   # not without dK
        assert rule("dq", STUDENT, 192, 64, heads, nq, nk, True) == rule("dk", STUDENT, 192, 64, heads, nq, nk, True) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("s1,s2,factor", EXTREME_SCALES)
def test_masked_pairs_at_extreme_scales(gpu_lib, s1, s2, factor):
    """The header admits every finite scale above 0. At these the stand-in for a masked logit would be of the order of
    the logits (a masked key then takes part) or overflow (0 x inf); backward on statistics computed elsewhere."""
    d = inputs.make("tiny", B=1, H=2, n_q=600, n_k=600, s1=s1, s2=s2)
    for n in ("Q1", "K1", "Q2", "K2"):
        d[n] = d[n] * np.float32(factor)   # exact in bf16
    kl, lse1, lse2, *ref = oracle.backward(d["Q1"], d["K1"], d["Q2"], d["K2"], s1, s2, True, 0, d["g"])
    got = gpu_lib.bwd(*upload(d), *(to_gpu_f32(x) for x in (kl, lse1, lse2, d["g"])), s1, s2, True, 0, want=ALL)
    for n, x, r in zip(ALL, got, ref):
        check_grad(n, x.cpu().numpy(), r)


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", ["dq", "dk"])
def test_reach_of_a_nonfinite_row_with_two_blocks(gpu_lib, kernel):
    """A wave's tiles serve its 64 resident rows: an infinity in column 5 of a streamed row can reach column 5 of the
    gradients of the wave's rows that it does not take part in (0 x inf), and nothing else. The rest of the head and the
    other heads keep their bits."""
    import torch
    heads, nq, nk = 32, 16400, 16400
    gen = torch.Generator(device="cuda").manual_seed(5)
    t = [torch.randn(1, heads, n, d, generator=gen, device="cuda", dtype=torch.bfloat16)
         for n, d in ((nq, 128), (nk, 128), (nq, 64), (nk, 64))]

    def grad():
        stats = gpu_lib.fwd(*t, causal=True)
        return gpu_lib.bwd(*t, *stats, causal=True, want=STUDENT)[2 if kernel == "dq" else 3]

    clean = grad()
    at = 170 if kernel == "dq" else 4010   # of 64-row waves [128, 192) and [3968, 4032)
    if kernel == "dq":
        t[3][0, 3, nk - nq + at, 5] = float("inf")   # a key that rows from 170 on see
        apart, seen = slice(0, 128), slice(128, at)
    else:
        t[2][0, 3, at, 5] = float("inf")             # a row that keys 0 to 4010 are seen by
        apart, seen = slice(4032, nk), slice(at + 1, 4032)
    bad = grad()
    assert not torch.isfinite(bad[0, 3, at]).all()
    assert torch.equal(clean[0, 3, apart], bad[0, 3, apart])
    cols = [c for c in range(64) if c != 5]
    assert torch.equal(clean[0, 3, seen][:, cols], bad[0, 3, seen][:, cols])
    clean[0, 3], bad[0, 3] = 0.0, 0.0
    assert torch.equal(clean, bad)


def test_reach_is_tested_on_two_blocks(rule):
    assert rule("dq", STUDENT, 128, 64, 32, 16400, 16400, True) == rule("dk", STUDENT, 128, 64, 32, 16400, 16400, True) == 2

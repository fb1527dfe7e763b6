"""The pipelined backward kernels: they compile without spilling, and they give the gradients of the plain kernels bit for
bit. A head's gradients do not depend on how many heads a call holds, while the kernel that computes them does: at most
256 workgroups of 128 rows take the pipelined form with one row block per wave, more take the plain one, and many
workgroups of 256 rows the pipelined form with two."""
import concurrent.futures as cf
import re
import subprocess

import pytest

from paper_2606_20005_amd import build

ALL = ("dq1", "dk1", "dq2", "dk2")


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


@pytest.mark.gpu
@pytest.mark.parametrize("heads,nq,nk,causal", [
    (512, 70, 16400, False), (512, 70, 16400, True), (512, 1, 16385, False),   # two blocks for dQ
    (520, 4101, 70, False), (1024, 8200, 33, True), (1024, 8300, 290, True),   # two blocks for dK
])
@pytest.mark.parametrize("d1,d2,want", [(128, 128, ("dq2", "dk2")), (128, 64, ("dq2", "dk2")), (64, 128, ("dq2", "dk2")),
                                        (128, 64, ("dq1", "dk1")), (64, 64, ("dq2", "dk2")), (64, 64, ALL)])
def test_same_bits_at_every_grid_size(gpu_lib, heads, nq, nk, causal, d1, d2, want):
    """Ragged tiles, one-row tiles, rows without keys, negative and zero upstream gradients. (64, 64) and all four
    gradients have no form with two blocks."""
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
    for lo, hi in ((0, 300), (5, 35)):   # the plain kernels; one block
        for a, b in zip(whole, grads(lo, hi)):
            assert torch.isfinite(b).all()
            assert torch.equal(a[:, lo:hi], b), (lo, hi)


@pytest.mark.gpu
@pytest.mark.parametrize("d1,d2,want", [(256, 64, ("dq2", "dk2")), (192, 128, ("dq2", "dk2")), (256, 256, ("dq1", "dk1")),
                                        (128, 128, ALL), (64, 192, ALL), (64, 256, ("dq1", "dk1"))])
@pytest.mark.parametrize("nq,nk,causal", [(130, 200, True), (40, 33, False)])
def test_wide_heads_key_gradients_match_the_plain_kernel(gpu_lib, d1, d2, want, nq, nk, causal):
    """Where the pipelined kernels run at every size: dK without a dQ in the call takes the plain kernel, which forms
    the row statistics itself."""
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

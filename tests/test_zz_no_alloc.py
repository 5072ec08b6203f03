"""The no-allocation projection (galore_project_noalloc) against the same
projection with a caller workspace (galore_project), through the C ABI, run
with -m gpu: two calls in a row, the second with a smaller input, in both
orientations; the results are bit-identical (same kernels, the scratch only
moves into the library's own device array), and sampled entries are checked
against host fp64 at the projection's tolerance (|x - ref| <= 1e-6 + 1e-5 |ref|)."""
import numpy as np
import pytest

import galore_inputs as gi
from metrics import max_rel_violation

pytestmark = pytest.mark.gpu


def _orthonormal(b, s, r, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    z = torch.randn((b, s, r), generator=g, device="cuda")
    return torch.linalg.qr(z)[0].contiguous()


@pytest.mark.parametrize("shapes", [((4096, 11008, 1024, 2), (1024, 2752, 256, 3)),
                                    ((11008, 4096, 1024, 2), (2736, 1024, 256, 1))])
def test_project_noalloc_equals_workspace_call(shapes):
    import torch
    import paper_2504_20437_amd as gl
    for call, (m, n, r, B) in enumerate(shapes):
        s, l = min(m, n), max(m, n)
        print("no-alloc projection call %d: %d x %dx%d r=%d" % (call, B, m, n, r), flush=True)
        G = gi.torch_planted_group(m, n, B, gi.spectrum_power(s, 0.7), 1e-4, seed=7000 + call, dtype="bf16")
        P = _orthonormal(B, s, r, 7100 + call)
        R_ws = gl.galore_project(P, G)                        # caller workspace (allocated by the binding)
        R_na = torch.full((B, r, l), float("nan"), device="cuda")
        gl.galore_project_noalloc(P, G, R_na)
        torch.cuda.synchronize()
        assert torch.equal(R_na, R_ws)
        rng = np.random.default_rng(call)
        ii, jj = rng.integers(0, r, 48), rng.integers(0, l, 48)
        for b in range(B):
            Pb = P[b].double().cpu().numpy()
            A = G[b].double().cpu().numpy()
            A = A if m <= n else A.T
            ref = np.array([Pb[:, i] @ A[:, j] for i, j in zip(ii, jj)])
            got = R_na[b].double().cpu().numpy()[ii, jj]
            assert max_rel_violation(got, ref, 1e-5, 1e-6) <= 1.0


@pytest.mark.parametrize("m,n,r,B", [
    (2048, 5461, 512, 1),        # planes and copy of one matrix fit the library's array
    (2048, 5461, 512, 8),        # ... of the batch do not: matrices at a time (2, 2, 2, 2)
    (300, 9001, 64, 37),         # ... an odd number of them
    (5461, 2047, 300, 5),
    (4097, 11007, 1024, 1),      # not even one copy: pieces along l, the last one short
    (11007, 4097, 1024, 2),
    (24, 3000, 4, 3),            # thin and small: the fp32 matrix cores in either call
])
def test_project_noalloc_ragged_equals_workspace_call(m, n, r, B):
    """bf16 gradients off the 16-byte grid: the same bits as with a workspace, in
    any batch, and sampled entries of the first and last matrix against fp64 to
    the fp32 bound (s 2^-24 of the sum of the products' sizes and a few ulps)."""
    import torch
    import paper_2504_20437_amd as gl
    s, l = min(m, n), max(m, n)
    gen = torch.Generator(device="cuda").manual_seed(m + n + B)
    G = torch.randn((B, m, n), generator=gen, device="cuda").to(torch.bfloat16)
    P = torch.randn((B, s, r), generator=gen, device="cuda")
    R = torch.full((B, r, l + 3), float("nan"), device="cuda")
    out = R[:, :, :l]
    gl.galore_project_noalloc(P, G, out)
    assert torch.equal(out, gl.galore_project(P, G))
    assert bool(R[:, :, l:].isnan().all())
    one = torch.empty((r, l), device="cuda")
    gl.galore_project_noalloc(P[B - 1], G[B - 1], one)
    assert torch.equal(one, out[B - 1])
    cols = torch.randint(0, l, (64,), generator=gen, device="cuda")
    cols[:3] = torch.tensor([0, l - 1, l // 2], device="cuda")
    for b in {0, B - 1}:
        A = (G[b] if m <= n else G[b].T).index_select(1, cols).double().contiguous()
        Pt = P[b].double().T.contiguous()
        bound = (s * 2.0 ** -24 + 2.0 ** -22) * (Pt.abs() @ A.abs())
        assert bool(((out[b].index_select(1, cols).double() - Pt @ A).abs() <= bound).all())

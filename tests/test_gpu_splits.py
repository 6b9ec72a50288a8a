"""Launches whose contraction is split over workgroups, at the sizes where the split changes: the
Coulomb build over P (none below 8 rows, at most 128 splits, pairs around its 1024-pair tile).

Bar: 1e-10 normwise against the FP64 oracle, as in test_gpu_parity.py (reordering a sum of at most
1e6 terms costs about 1e-13)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import df_grad as G
from oracle import df_oracle as O
from paper_2505_03755_amd import dfmi, synth

pytestmark = pytest.mark.gpu
TOL = 1e-10


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda")


def close(gpu, ref, what=""):
    g, r = gpu.detach().cpu().numpy(), np.asarray(ref, dtype=np.float64)
    assert g.shape == r.shape, what
    assert np.isfinite(g).all(), what
    assert np.linalg.norm(g - r) <= TOL * np.linalg.norm(r), (what, np.linalg.norm(g - r) / np.linalg.norm(r))
    assert np.abs(g - r).max() <= TOL * np.abs(r).max(), what


# nao 44 / 45: 990 / 1035 packed pairs; naux 7 / 8: no split / two; 600: the 128-split cap
@pytest.mark.parametrize("nao,naux,ndm", [(44, 8, 1), (45, 7, 2), (45, 9, 3), (3, 600, 4), (91, 257, 5), (1, 1, 1)])
@pytest.mark.parametrize("weighted", [False, True])
def test_jk_coulomb_splits(nao, naux, ndm, weighted):
    rng = np.random.default_rng(nao * 1000 + naux)
    nocc = max(1, nao // 4)
    B = rng.standard_normal((naux, O.npair(nao)))
    C = rng.standard_normal((ndm, nao, nocc))
    w = rng.standard_normal((ndm, nocc)) if weighted else None
    gB, gC, gw = dev(B), dev(C), dev(w) if weighted else None
    J, K, v = dfmi.jk(gB, nao, gC, w=gw)
    out = {"J": torch.ones_like(J), "K": torch.ones_like(K), "v": torch.ones_like(v)}
    dfmi.jk(gB, nao, gC, w=gw, out=out, accumulate=True)
    nal = {k: torch.empty_like(t) for k, t in (("J", J), ("K", K), ("v", v))}
    dfmi.jk_noalloc(gB, nao, gC, w=gw, out=nal)
    torch.cuda.synchronize()
    for z in range(ndm):
        Jr, Kr, vr = O.jk(B, nao, C[z], None if w is None else w[z])
        for name, got, ref in (("J", J, Jr), ("K", K, Kr), ("v", v, vr)):
            close(got[z], ref, f"{name}[{z}]")
            close(nal[name][z], ref, f"no-allocation {name}[{z}]")
            close(out[name][z], 1.0 + ref, f"accumulated {name}[{z}]")
    assert torch.equal(J, J.transpose(1, 2))


@pytest.mark.parametrize("nao,naux", [(33, 40), (120, 480)])
def test_adjoint_coulomb_under_scratch_limit(nao, naux):
    """The adjoint's Coulomb part takes its partial sums from the pieces a scratch limit leaves."""
    nocc, nac = nao // 4, 4
    B = synth.cholesky_vectors(naux, nao, 10.0, seed=3)
    C = synth.orbitals(nao, seed=3)
    Co, Ca = C[:, :nocc].copy(), C[:, nocc:nocc + nac].copy()
    rng = np.random.default_rng(5)
    gJ, gK, ge = rng.standard_normal((nao, nao)), rng.standard_normal((nao, nao)), rng.standard_normal((nac,) * 4)
    ctx = dfmi.Context()
    for cot in ((gJ, None, None), (gJ, gK, ge)):
        ref = G.step_vjp(B, nao, Co, Ca, *cot)
        flags = sum(f for f, c in zip((dfmi.DF_BWD_GJ, dfmi.DF_BWD_GK, dfmi.DF_BWD_GERI), cot) if c is not None)
        for limit in (0, 1):
            ctx.set_scratch_limit(0)
            if limit:   # the smallest bound: one auxiliary row per chunk
                lo, hi = 1, ctx.workspace_query(dfmi.DF_OP_STEP_BACKWARD, naux=naux, nao=nao, ndm=1, nocc=nocc,
                                                nac=nac, flags=flags)
                while lo < hi:
                    mid = (lo + hi) // 2
                    ctx.set_scratch_limit(mid)
                    try:
                        ctx.backward_chunk(naux=naux, nao=nao, ndm=1, nocc=nocc, nac=nac, flags=flags)
                        hi = mid
                    except dfmi.DFError:
                        lo = mid + 1
                ctx.set_scratch_limit(lo)
                ctx.release_workspace()
            g = [None if c is None else dev(c) for c in cot]
            dCo, dCa = dfmi.step_backward(dev(B), nao, dev(Co), dev(Ca), *g, ctx=ctx)
            torch.cuda.synchronize()
            close(dCo, ref[0], f"dCocc limit {limit}")
            if cot[2] is not None:
                close(dCa, ref[1], f"dCact limit {limit}")

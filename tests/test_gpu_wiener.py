"""Nonstationary Wiener deblurring (appendix D) on the GPU (hipFFT), through
the C ABI, against the FP64 oracle (numpy FFT).

Bar: FP32 transforms of tapered blocks followed by a regularised division;
relative L2 error 1e-4 against the FP64 oracle, as for the operators.
"""
import numpy as np
import pytest

from oracle import lsrtm_oracle as O
from paper_2508_10405_amd import synth
from gpu_common import f64, oracle_problem, rel, require_gpu, to_dev

pytestmark = pytest.mark.gpu
TOL = 1e-4


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


CASES = [((37, 45), 16, 1e-3), ((64, 75), 32, 1e-2), ((240, 100), 64, 1e-3), ((12, 14, 10), 8, 1e-3),
         # blocks larger than the image along every axis
         ((20, 24), 64, 1e-3), ((5, 6, 4), 8, 1e-3)]


@pytest.mark.parametrize("n,block,eps", CASES)
def test_wiener_vs_oracle_random(torch, n, block, eps):
    from paper_2508_10405_amd import lsrtm
    print(f"[case] wiener {n} block {block} eps {eps}", flush=True)
    shape = tuple(reversed(n))
    ctx = lsrtm.Context(n, (10.0,) * len(n), 10, 1e-3)
    rng = np.random.default_rng(sum(n) + block)
    ref, blur, x = (rng.standard_normal(shape) for _ in range(3))
    out = ctx.wiener(to_dev(torch, ref), to_dev(torch, blur), to_dev(torch, x), block=block, eps_rel=eps)
    expect = O.wiener_deblur(ref, blur, x, block, eps)
    e = rel(out.cpu().numpy(), expect)
    print("wiener rel", e, flush=True)
    assert e <= TOL
    ctx.close()


def test_wiener_identity(torch):
    """Unregularised filter of an image by itself is the identity."""
    from paper_2508_10405_amd import lsrtm
    n = (50, 61)
    ctx = lsrtm.Context(n, (10.0, 10.0), 10, 1e-3)
    rng = np.random.default_rng(7)
    m = to_dev(torch, rng.standard_normal((61, 50)))
    x = to_dev(torch, rng.standard_normal((61, 50)))
    out = ctx.wiener(m, m, x, block=16, eps_rel=0.0)
    e = rel(out.cpu().numpy(), x.cpu().numpy())
    print("identity rel", e, flush=True)
    assert e <= 1e-5
    ctx.close()


def test_wiener_on_migrated_images(torch):
    """The paper's use: m_ref = m_in = RTM image, m_blur = its remigration
    L^T L m_rtm, both parameters in one call (each filtered on its own)."""
    from paper_2508_10405_amd import lsrtm
    w = synth.small((48, 64), nt=140, npml=8, seed=61, nshot=3, uneven=True)
    ctx = lsrtm.context_for(w)
    m_rtm = ctx.adjoint(ctx.born(to_dev(torch, w.dm)))
    m_rem = ctx.adjoint(ctx.born(m_rtm))
    out = ctx.wiener(m_rtm, m_rem, block=16, eps_rel=1e-3)
    for k in range(2):
        expect = O.wiener_deblur(m_rtm[k].cpu().numpy().astype(np.float64),
                                 m_rem[k].cpu().numpy().astype(np.float64),
                                 m_rtm[k].cpu().numpy().astype(np.float64), 16, 1e-3)
        e = rel(out[k].cpu().numpy(), expect)
        print("migrated wiener", k, e, flush=True)
        assert e <= TOL
    single = ctx.wiener(m_rtm[1].contiguous(), m_rem[1].contiguous(), block=16, eps_rel=1e-3)
    assert torch.equal(single, out[1])
    ctx.close()
    # oracle-only chain: the oracle's RTM image and remigration, then its filter
    prob = oracle_problem(w)
    lnvp, lnip = f64(w.lnvp), f64(w.lnip)
    LtL = lambda m: O.adjoint(prob, lnvp, lnip, O.born(prob, lnvp, lnip, m))
    r_rtm = LtL(f64(w.dm))
    r_rem = LtL(r_rtm)
    for k in range(2):
        expect = O.wiener_deblur(r_rtm[k], r_rem[k], r_rtm[k], 16, 1e-3)
        e = rel(out[k].cpu().numpy(), expect)
        print("migrated wiener, oracle-only chain", k, e, flush=True)
        assert e <= TOL


def test_wiener_errors(torch):
    from paper_2508_10405_amd import lsrtm
    ctx = lsrtm.Context((20, 24), (10.0, 10.0), 10, 1e-3)
    m = torch.zeros((24, 20), device="cuda")
    for block, eps in ((15, 1e-3), (0, 1e-3), (16, -1.0)):
        with pytest.raises(lsrtm.LsrtmError):
            ctx.wiener(m, m, block=block, eps_rel=eps)
    ctx.close()


@pytest.mark.parametrize("block", [16, 32, 64])
def test_wiener_stacks(torch, block):
    """A stack of more images than a launch takes, sizes that are no multiple
    of the block, m_in given and left out: each image as by a call of its own,
    and as the oracle has it (the operators' bar, as above)."""
    from paper_2508_10405_amd import lsrtm
    n, k = (71, 37), 5
    rng = np.random.default_rng(block)
    ctx = lsrtm.Context(n, (10.0, 10.0), 10, 1e-3)
    ref, blur, x = (rng.standard_normal((k, 37, 71)) * 10.0 ** rng.uniform(-12, 3, (k, 1, 1)) for _ in range(3))
    d = [to_dev(torch, v) for v in (ref, blur, x)]
    for third in (None, 2):
        out = ctx.wiener(d[0], d[1], None if third is None else d[third], block=block, eps_rel=1e-3)
        for i in range(k):
            own = ctx.wiener(*(v[i].contiguous() for v in d[:2]), None if third is None else d[third][i].contiguous(),
                             block=block, eps_rel=1e-3)
            assert torch.equal(own, out[i])
            expect = O.wiener_deblur(ref[i], blur[i], ref[i] if third is None else x[i], block, 1e-3)
            e = rel(out[i].cpu().numpy(), expect)
            print("wiener stack", block, third, i, e, flush=True)
            assert e <= TOL
    ctx.close()


@pytest.mark.parametrize("block", [16, 32, 64, 24])
def test_wiener_under_capture(torch, block):
    """After a first call of one image, a stack of five is captured into a
    graph (nothing is allocated any more); its replays, with eager calls of
    other stacks between them, give the eager result for the inputs of the
    moment."""
    from paper_2508_10405_amd import lsrtm
    n, k = (71, 37), 5
    g = torch.Generator(device="cuda").manual_seed(block)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        ctx = lsrtm.Context(n, (10.0, 10.0), 10, 1e-3)
        ref, blur = (torch.randn((k, 37, 71), generator=g, device="cuda") for _ in range(2))
        ctx.wiener(ref[0].contiguous(), blur[0].contiguous(), block=block)
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            out = ctx.wiener(ref, blur, block=block)
        for _ in range(3):
            ref.copy_(torch.randn((k, 37, 71), generator=g, device="cuda"))
            graph.replay()
            got = out.clone()
            assert torch.equal(got, ctx.wiener(ref, blur, block=block))
        st.synchronize()
    ctx.close()


@pytest.mark.parametrize("block", [16, 32, 64])
def test_wiener_nan_in_the_blurred_image(torch, block):
    """A NaN in m_blur takes the blocks that hold it out of the result (their
    estimates are zero) and touches nothing else."""
    from paper_2508_10405_amd import lsrtm
    n = (171, 137)
    g = torch.Generator(device="cuda").manual_seed(block)
    ctx = lsrtm.Context(n, (10.0, 10.0), 10, 1e-3)
    ref, blur, x = (torch.randn((137, 171), generator=g, device="cuda") for _ in range(3))
    clean = ctx.wiener(ref, blur, x, block=block)
    h = block // 2
    for at in ((0, 0), (70, 85), (136, 30), (64, 64), (h, 2 * h)):
        bad = blur.clone()
        # the largest magnitude scales the image: not that one
        assert float(bad[at].abs()) < float(bad.abs().max())
        bad[at] = float("nan")
        out = ctx.wiener(ref, bad, x, block=block)
        assert bool(torch.isfinite(out).all()), at
        # blocks start at (k - 1) h: those with the NaN are k = c / h and c / h + 1 per axis
        near = torch.zeros_like(out, dtype=torch.bool)
        kx, kz = at[0] // h, at[1] // h
        near[max(0, (kx - 1) * h):(kx + 2) * h, max(0, (kz - 1) * h):(kz + 2) * h] = True
        assert torch.equal(out[~near], clean[~near]), at
        assert not bool(out[kx * h:(kx + 1) * h, kz * h:(kz + 1) * h].any()), at
    ctx.close()

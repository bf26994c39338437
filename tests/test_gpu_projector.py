"""R_T and R_T* of the plain form at the edges of their work split, against the
FP64 oracle.

Tolerance 1e-5 of the result (rel-L2 and, scaled by the largest value, per
element): each value is a sum of up to 2 N K products of unit scale in FP32,
whose rounding is below 2^-24 sqrt(2 N K) of it, at most 1e-5 for the N and K
here, with the position's 2^-32 per line far below."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1809_09725_amd import inputs, rt4d

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


def geom(N, Nz, Ns, Npi, n0, K):
    return rt4d.Geom(N=N, Nz=Nz, Ns=Ns, Ntheta=Npi * n0, Npi=Npi, K=K, Nt=1)


CASES = [
    # channel quads per workgroup (1, 2, 4), quads of several slices, ragged
    # last quads, fewer than four channels
    geom(37, 1, 41, 2, 9, 1), geom(37, 2, 41, 2, 9, 3), geom(37, 5, 41, 2, 9, 2),
    geom(37, 1, 41, 2, 9, 4), geom(37, 1, 41, 2, 9, 5), geom(37, 3, 41, 2, 9, 7),
    geom(37, 3, 41, 2, 9, 8), geom(37, 2, 41, 2, 9, 12), geom(37, 2, 41, 2, 9, 15),
    geom(37, 2, 41, 2, 9, 18), geom(37, 1, 41, 2, 9, 33),
    # bin blocks of 64 and their tiles; detectors narrower and wider than the slice
    geom(64, 2, 63, 2, 13, 16), geom(64, 2, 64, 2, 13, 16), geom(64, 2, 65, 2, 13, 16),
    geom(90, 1, 700, 2, 40, 16), geom(300, 1, 20, 2, 24, 16),
    # many classes (full workgroups), one class, windows and whole lines
    geom(256, 24, 256, 2, 128, 4), geom(200, 40, 230, 2, 60, 16), geom(120, 1, 120, 3, 1, 16),
    geom(512, 1, 512, 2, 90, 16),
    # two-level sums: N > 512, with the flush every 64 lines inside parts
    geom(513, 2, 300, 2, 12, 8), geom(640, 1, 640, 2, 30, 15), geom(1023, 1, 520, 1, 6, 4),
    geom(1100, 1, 200, 2, 10, 16),
    # one position, one bin
    geom(1, 3, 1, 2, 4, 4), geom(2, 1, 130, 2, 5, 16),
]


@pytest.mark.parametrize("G", CASES, ids=lambda G: f"N{G.N}z{G.Nz}s{G.Ns}a{G.n0}k{G.K}")
def test_forward_edges(G):
    torch.cuda.set_device(DEV)
    print(f"case {G}", flush=True)
    f = inputs.uniform(G.f_shape, 5)
    got = rt4d.Plan(G).forward(torch.from_numpy(f).to(DEV)).cpu().numpy().astype(np.float64)
    want = O.forward(O.Geom(**G.__dict__), f)
    assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want)
    assert np.abs(got - want).max() <= 1e-5 * np.abs(want).max()


FEW_CHANNELS = [   # a quad per slice: 1, 2 and 4 slices per workgroup and a ragged last one, long lines, many classes
    geom(64, 9, 64, 3, 13, 1), geom(200, 7, 130, 2, 60, 3), geom(256, 20, 256, 2, 128, 2), geom(166, 5, 110, 18, 40, 2),
    geom(530, 6, 530, 2, 7, 1), geom(600, 1, 400, 1, 9, 2), geom(600, 3, 620, 2, 12, 3), geom(600, 2, 620, 20, 4, 3),
]


@pytest.mark.parametrize("G", FEW_CHANNELS, ids=lambda G: f"N{G.N}z{G.Nz}s{G.Ns}p{G.Npi}k{G.K}")
def test_forward_few_channels(G):
    """Fewer than four channels, at the same bar."""
    test_forward_edges(G)


MANY_HALF_TURNS = [   # contracted in parts of the half-turns, with and without line parts; in the projection, ragged last group
    geom(20, 2, 24, 40, 3, 20), geom(8, 5, 5, 34, 12, 45), geom(64, 1, 64, 20, 9, 8), geom(40, 3, 50, 17, 7, 6),
    geom(48, 15, 48, 13, 60, 7), geom(48, 16, 48, 16, 60, 4), geom(48, 7, 48, 9, 70, 16), geom(30, 9, 33, 5, 64, 3),
]


@pytest.mark.parametrize("G", MANY_HALF_TURNS, ids=lambda G: f"N{G.N}z{G.Nz}s{G.Ns}p{G.Npi}k{G.K}")
def test_forward_many_half_turns(G):
    """The contraction with Phi over many half-turns, at the same bar."""
    test_forward_edges(G)


PACKED_RAYS = [   # detectors of no whole number of ray blocks: blocks over two and more classes, in full and small workgroups,
    # fused with Phi, through line parts, per ragged quad and below four channels; half-turns of both directions of the bins
    geom(70, 1, 70, 2, 200, 16), geom(80, 40, 80, 3, 90, 8), geom(100, 30, 100, 2, 200, 7), geom(130, 12, 130, 3, 70, 4),
    geom(66, 40, 66, 18, 60, 16), geom(66, 5, 17, 5, 300, 2), geom(33, 50, 5, 3, 201, 16), geom(48, 40, 48, 8, 100, 15),
    geom(128, 20, 129, 2, 180, 16), geom(256, 20, 257, 2, 90, 8), geom(530, 2, 530, 2, 40, 12), geom(64, 12, 1, 4, 150, 20),
]


@pytest.mark.parametrize("G", PACKED_RAYS, ids=lambda G: f"N{G.N}z{G.Nz}s{G.Ns}a{G.n0}k{G.K}")
def test_forward_packed_rays(G):
    """Ray blocks over several classes, at the same bar."""
    test_forward_edges(G)


@pytest.mark.parametrize("G", [geom(3664, 1, 64, 1, 5, 20), geom(2048, 2, 90, 1, 5, 58)],
                         ids=lambda G: f"N{G.N}z{G.Nz}k{G.K}")
def test_forward_large_slices(G):
    """Quads of a slice whose offsets take more than 32 bits (through
    registers), and a list of quads over slices of 0.97 GB.  Lines of N > 512:
    2^-25 sqrt(32 + N / 64 + K / 2) of the result in rel-L2, as the rounding
    of two-level sums has it (line parts only lessen it)."""
    torch.cuda.set_device(DEV)
    print(f"case {G}", flush=True)
    f = inputs.uniform(G.f_shape, 9)
    got = rt4d.Plan(G).forward(torch.from_numpy(f).to(DEV)).cpu().numpy().astype(np.float64)
    want = O.forward(O.Geom(**G.__dict__), f)
    e = np.linalg.norm(got - want) / np.linalg.norm(want)
    print(f"rel-L2 {e:.3e}", flush=True)
    assert e <= 2.0 ** -25 * np.sqrt(32 + G.N / 64 + G.K / 2)
    assert np.abs(got - want).max() <= 1e-5 * np.abs(want).max()


ADJOINT_CASES = CASES + [
    # 32 x 32 tiles (the cases above fill few: 32 x 8), ragged and aligned,
    # quads of one and of several slices, a ragged last quad; detectors that end
    # inside the slice; more classes than one fill of the class table
    geom(128, 64, 128, 2, 5, 16), geom(100, 40, 60, 3, 9, 20), geom(97, 90, 140, 2, 7, 7),
    geom(40, 3, 30, 2, 131, 16), geom(33, 2, 500, 4, 65, 6), geom(31, 2, 8, 2, 64, 16),
]


@pytest.mark.parametrize("G", ADJOINT_CASES, ids=lambda G: f"N{G.N}z{G.Nz}s{G.Ns}a{G.n0}k{G.K}")
def test_adjoint_edges(G):
    """Each value sums at most 2 Ntheta products of unit scale (weights up to
    sqrt 2): the same bar."""
    torch.cuda.set_device(DEV)
    print(f"case {G}", flush=True)
    g = inputs.uniform(G.g_shape, 7)
    got = rt4d.Plan(G).adjoint(torch.from_numpy(g).to(DEV)).cpu().numpy().astype(np.float64)
    want = O.adjoint(O.Geom(**G.__dict__), g)
    assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want)
    assert np.abs(got - want).max() <= 1e-5 * np.abs(want).max()


@pytest.mark.parametrize("K", [4, 8, 11, 16])
def test_slices_do_not_depend_on_the_volume(K):
    """A slice's projections are the same bits whichever slices share its
    workgroup, and non-finite values stay in the slices that hold them."""
    torch.cuda.set_device(DEV)
    G = geom(96, 24, 100, 4, 64, K)
    f = torch.from_numpy(inputs.uniform(G.f_shape, 6)).to(DEV)
    p = rt4d.Plan(G)
    a = p.forward(f)
    f2 = f.clone()
    f2[3, 40, 40, 0] = float("nan")
    f2[9, 10, 50, K - 1] = float("inf")
    b = p.forward(f2)
    keep = [z for z in range(G.Nz) if z not in (3, 9)]
    assert torch.equal(a[:, keep], b[:, keep])
    assert torch.isnan(b[:, 3]).any() and not torch.isnan(b[:, 3]).all()
    assert not torch.isfinite(b[:, 9]).all()
    g = torch.from_numpy(inputs.uniform(G.g_shape, 8)).to(DEV)
    a = p.adjoint(g)
    g2 = g.clone()
    g2[5, 3, 50] = float("nan")
    g2[70, 9, 20] = float("inf")
    b = p.adjoint(g2)
    assert torch.equal(a[keep], b[keep])
    assert torch.isnan(b[3]).any() and not torch.isnan(b[3]).all()
    assert not torch.isfinite(b[9]).all()


@pytest.mark.parametrize("N", [513, 640, 1024])
def test_two_level_sums_rounding(N):
    """Lines of more than 512 positions in one part (the workgroups fill the
    chip), signed data, where rounding errors add as a random walk.  A sum of
    terms of unit size over blocks of L lines, kept one rounding per addition
    and blocks added likewise, collects the variance sum of l over each block
    (N L / 2 in all, N L with two roundings per line) plus N^2 / (2 L) of the
    block sums, in units of the terms' variance and of a rounding's, whose rms
    is below 2^-25 of the value (half a unit roundoff); K channels contracted
    add K / 2.  Blocks of 32 lines with two roundings, relative to the N of the
    sum: 2^-25 sqrt(32 + N / 64 + K / 2)."""
    torch.cuda.set_device(DEV)
    G = geom(N, 32, N, 1, 300, 4)
    f = torch.zeros(G.f_shape, device=DEV)
    zs = (0, 13, 30)
    host = {z: inputs.uniform((N, N, 4), 40 + z) for z in zs}
    for z in zs:
        f[z] = torch.from_numpy(host[z]).to(DEV)
    got = rt4d.Plan(G).forward(f)
    num = den = 0.0
    for z in zs:
        want = O.forward(O.Geom(**{**G.__dict__, "Nz": 1}), host[z][None])[:, 0]
        num += float(np.sum((got[:, z].cpu().numpy().astype(np.float64) - want) ** 2))
        den += float(np.sum(want ** 2))
    bound = 2.0 ** -25 * np.sqrt(32 + N / 64 + 4 / 2)
    print(f"N {N}: rel-L2 {np.sqrt(num / den):.3e} (bound {bound:.3e})", flush=True)
    assert np.sqrt(num / den) <= bound


SF_CASES = [   # (geometry): slots per group 4, 2, 1 and 1, 2, 4 bins of 512 per slot; 16..64 channels
    geom(37, 2, 41, 2, 9, 4), geom(64, 1, 64, 8, 7, 16), geom(33, 1, 60, 9, 6, 20), geom(31, 2, 30, 16, 5, 33),
    geom(65, 1, 70, 17, 4, 40), geom(40, 1, 44, 27, 3, 64), geom(96, 1, 90, 32, 4, 64), geom(1, 2, 1, 3, 4, 7),
    geom(400, 1, 400, 8, 5, 16), geom(257, 2, 256, 4, 4, 24), geom(256, 1, 256, 8, 4, 16),
    # lines of two and more chunks, with a few positions in the last one; one chunk exactly
    geom(512, 1, 520, 4, 5, 8), geom(513, 1, 700, 8, 6, 32), geom(545, 1, 900, 12, 4, 24), geom(1030, 1, 300, 16, 3, 17),
    geom(200, 1, 1300, 8, 5, 16), geom(150, 1, 2048, 12, 4, 30), geom(130, 1, 1100, 20, 3, 20), geom(90, 1, 2100, 4, 4, 64),
]


@pytest.mark.parametrize("G", SF_CASES, ids=lambda G: f"N{G.N}z{G.Nz}s{G.Ns}p{G.Npi}k{G.K}")
def test_synthesise_first_edges(G):
    """Volumes on the BF16 grid, so that only Phi's two BF16 parts (within
    2^-17 of a value of at most 1) and FP32 sums over 2 N taps round, both
    relative to S, the projection of sum_k |f_k|, and the positions, within
    2^-32 (1 + l) on line l: below N^2 2^-31 of the largest sum_k |f_k| over
    the lines (the angle pi is not exact in the oracle: rays that just miss the
    slice have S near 1e-14 there)."""
    torch.cuda.set_device(DEV)
    print(f"case {G}", flush=True)
    f = torch.from_numpy(inputs.uniform(G.f_shape, 8)).to(torch.bfloat16).to(torch.float32)
    p = rt4d.Plan(G, form=rt4d.RT_FORM_SF, prec=rt4d.RT_PREC_BF16MFMA)
    got = p.forward(f.to(DEV)).cpu().numpy().astype(np.float64)
    want = O.forward(O.Geom(**G.__dict__), f.numpy())
    G1 = O.Geom(**{**G.__dict__, "K": 1})
    F = f.abs().sum(-1, keepdim=True).numpy()
    S = O.forward(G1, F)
    assert (np.abs(got - want) <= (2.0 ** -17 + 4 * G.N * 2.0 ** -24) * S + G.N ** 2 * 2.0 ** -31 * F.max()).all()


SF_WIDE = [   # 33..64 channels over more than 512 bins
    geom(311, 1, 561, 20, 2, 39), geom(100, 1, 1300, 12, 3, 40), geom(70, 1, 1400, 4, 3, 48), geom(520, 1, 600, 13, 3, 52),
    geom(130, 1, 900, 32, 2, 64), geom(600, 1, 600, 5, 3, 58),
    geom(120, 1, 1400, 28, 2, 44), geom(300, 1, 700, 5, 4, 58), geom(257, 1, 1100, 12, 2, 64),
]


@pytest.mark.parametrize("G", SF_WIDE, ids=lambda G: f"N{G.N}s{G.Ns}p{G.Npi}k{G.K}")
def test_synthesise_first_many_channels(G):
    """The thread counts above 32 channels, at the same bar."""
    test_synthesise_first_edges(G)


SF_CHUNKS = [   # one chunk of 640 threads, of 768 (and three bins of them), two of 1024; ragged ends of lines in each
    geom(257, 1, 257, 9, 4, 16), geom(320, 1, 320, 20, 3, 24), geom(321, 2, 330, 28, 2, 7), geom(384, 1, 384, 16, 3, 32),
    geom(290, 1, 700, 28, 3, 33), geom(300, 2, 290, 16, 3, 60), geom(318, 1, 1100, 8, 3, 40), geom(383, 1, 500, 4, 5, 64),
    geom(350, 1, 1500, 4, 4, 48), geom(340, 1, 780, 32, 2, 50), geom(385, 1, 600, 12, 3, 40), geom(410, 1, 410, 8, 3, 64),
]


@pytest.mark.parametrize("G", SF_CHUNKS, ids=lambda G: f"N{G.N}s{G.Ns}p{G.Npi}k{G.K}")
def test_synthesise_first_line_chunks(G):
    """Lines of 257 to 512 positions, at the same bar."""
    test_synthesise_first_edges(G)

"""The measurement aids of the C ABI on the GPU: the FMA issue-rate kernel
(rt_calib_fma) against an FP32 emulation of its chains on the host, and the
per-kernel timing counters (rt_timing_*) around a forward projection."""
import numpy as np
import pytest
import torch

from paper_1809_09725_amd import inputs, rt4d

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


def test_calib_fma_chains_and_flop_count():
    torch.cuda.set_device(DEV)
    nb, it = 4, 3
    out = torch.empty(nb * 256, device=DEV)
    ms, flop = rt4d.calib_fma(nb, it, out)
    assert ms > 0.0
    assert flop == 2.0 * 8 * 16 * it * 256 * nb
    # eight chains x <- fma(x, 0.999, 0.001) from x = thread + chain, 16 per
    # iteration, summed in chain order; each fma rounds once to FP32 (the
    # FP64 product of two floats is exact, so only the final rounding counts
    # except in rare double-rounding cases: compared to 2 ulp)
    a, b = np.float32(0.999), np.float32(0.001)
    tid = np.arange(256, dtype=np.float64)
    s = np.zeros(256, np.float32)
    for c in range(8):
        x = (tid + c).astype(np.float32)
        for _ in range(16 * it):
            x = (x.astype(np.float64) * np.float64(a) + np.float64(b)).astype(np.float32)
        s = (s + x).astype(np.float32)
    got = out.cpu().numpy().reshape(nb, 256)
    for blk in range(nb):
        np.testing.assert_allclose(got[blk], s, rtol=2.5e-7, atol=0)


def test_timing_counters_around_a_forward():
    torch.cuda.set_device(DEV)
    G = rt4d.Geom(N=48, Nz=2, Ns=50, Ntheta=4 * 30, Npi=4, K=6, Nt=4)
    plan = rt4d.Plan(G)
    f = torch.from_numpy(inputs.uniform(G.f_shape, 5)).to(DEV)
    rt4d.timing_reset()
    rt4d.timing_enable(True)
    plan.forward(f)
    plan.forward(f)
    torch.cuda.synchronize()
    rt4d.timing_enable(False)
    ms, n = rt4d.timing_read("k_project")
    assert n == 2 and ms > 0.0
    plan.forward(f)   # not counted while disabled
    torch.cuda.synchronize()
    assert rt4d.timing_read("k_project")[1] == 2
    assert rt4d.timing_read("no_such_kernel") == (0.0, 0)
    rt4d.timing_reset()
    assert rt4d.timing_read("k_project") == (0.0, 0)
    plan.close()


@pytest.mark.parametrize("sf,dims", [
    (False, dict(N=16, Nz=1, Ns=2048, n0=3000, Npi=1, K=1)),      # many bins and classes: ray groups
    (False, dict(N=32, Nz=1, Ns=91, n0=16000, Npi=1, K=1)),       # many classes: class lists
    (True, dict(N=32, Nz=2, Ns=100, n0=9000, Npi=1, K=2)),
    (False, dict(N=8, Nz=512, Ns=2048, n0=300, Npi=1, K=1)),      # more than 2^18 partial sums
    (False, dict(N=64, Nz=3, Ns=91, n0=90, Npi=8, K=7)), (True, dict(N=128, Nz=1, Ns=128, n0=60, Npi=4, K=16)),
])
def test_job_bytes_cover_the_plan(sf, dims):
    """rt_job_bytes, the admission's figure, is at least what the plan holds
    and a job's state ((2 f + 2 g + 5 frames) floats) take."""
    torch.cuda.set_device(DEV)
    n0 = dims.pop("n0")
    G = rt4d.Geom(Ntheta=dims["Npi"] * n0, Nt=1, **dims)
    form = (rt4d.RT_FORM_SF, rt4d.RT_PREC_BF16MFMA) if sf else (rt4d.RT_FORM_PF, rt4d.RT_PREC_FP32)
    plan = rt4d.Plan(G, *form)
    nv = G.Nz * G.N * G.N
    state = 4 * (2 * nv * G.K + 2 * G.Ntheta * G.Nz * G.Ns + 5 * nv * G.Nt)
    print(f"{G}: plan {plan.bytes} + state {state}, rt_job_bytes {rt4d.rt_job_bytes(G, *form)}", flush=True)
    assert plan.bytes + state <= rt4d.rt_job_bytes(G, *form)
    plan.close()

"""Several parameter points side by side in one pass of the one-event-per-wave
kernels, and the split of a small batch's points over waves: each weight must be
what its point gives alone, whatever its place in the pass, the number of
points and the size of the batch.

Single precision: bit for bit (a point's amplitude is rounded as in the program
for one point).  Double precision: both results are held to 1e-12 of the
oracle, so they agree to 2e-12."""
import numpy as np
import pytest

from synth import generate_events, kappa_points

pytestmark = pytest.mark.gpu
FP64_TOL = 2e-12


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def handle(prec, npts, tau=None):
    import paper_2312_07440_amd as mg
    p = mg.Process("gg_ttgg", prec)
    kap = kappa_points(npts)
    p.set_params([{"kappa_ttg": float(k), "alphas": 0.118 * (1 + 0.01 * (i % 3))} for i, k in enumerate(kap)])
    if tau is not None:
        p.set_rescue_threshold(tau)
    return p


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("npts", [1, 2, 3, 4, 5, 16, 64])
@pytest.mark.parametrize("n", [1, 67])
def test_every_point_as_alone(torch_dev, prec, npts, n):
    torch = torch_dev
    mom = torch.from_numpy(generate_events("gg_ttgg", n, first_event=3 * 10 ** 5)).cuda()
    p = handle(prec, npts, 0.0 if prec == "mixed" else None)
    w_in = torch.linspace(0.5, 2.0, n, dtype=torch.float64, device="cuda")
    me0 = torch.empty(n, dtype=torch.float64, device="cuda")
    out = p.reweight(mom, w_in=w_in, me_base_out=me0)
    base = p.eval_me(mom)
    ref = torch.stack([w_in * (p.eval_me(mom, point=k) / base) for k in range(npts)])
    if prec == "mixed":
        assert torch.equal(out, ref) and torch.equal(me0, base)
    else:
        assert (out / ref - 1).abs().max() <= FP64_TOL and (me0 / base - 1).abs().max() <= FP64_TOL


@pytest.mark.parametrize("prec,tau", [("mixed", None), ("fp64", None), ("mixed", 1.0)])
@pytest.mark.parametrize("n", [16383, 16384, 16387])
def test_batch_size_does_not_matter(torch_dev, prec, tau, n):
    """Both sides of the size from which on a wave takes a whole event (with
    tau = 1 every event is re-evaluated in double precision, so the list of
    those has the same sizes)."""
    torch = torch_dev
    mom = torch.from_numpy(generate_events("gg_ttgg", n, first_event=10 ** 6)).cuda()
    p = handle(prec, 2, tau)
    out = p.reweight(mom)
    for sel in (slice(0, 131), slice(n - 70, n)):
        part = p.reweight(mom[:, :, sel].contiguous())
        assert torch.equal(out[:, sel], part)
    if tau == 1.0:
        ref = handle("fp64", 2).reweight(mom)
        assert (out / ref - 1).abs().max() <= FP64_TOL


@pytest.mark.parametrize("call", ["reweight", "reweight_noalloc"])
def test_weights_in_place(torch_dev, call):
    """The output may be the input weights' own buffer."""
    torch = torch_dev
    n = 300
    mom = torch.from_numpy(generate_events("gg_ttgg", n, first_event=77)).cuda()
    p = handle("mixed", 2)
    w = torch.linspace(0.5, 2.0, n, dtype=torch.float64, device="cuda")
    ref = p.reweight(mom, w_in=w)
    for row in (0, 1):
        buf = torch.zeros(2, n, dtype=torch.float64, device="cuda")
        buf[row] = w
        getattr(p, call)(mom, w_in=buf[row], out=buf)
        assert torch.equal(buf, ref)


def split_handle(prec, npts, tau=None):
    import paper_2312_07440_amd as mg
    p = mg.Process("gg_ttggg", prec)
    p.set_params([{"kappa_ttg": float(k), "alphas": 0.118 * (1 + 0.01 * (i % 3))}
                  for i, k in enumerate(kappa_points(npts))])
    if tau is not None:
        p.set_rescue_threshold(tau)
    return p


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("npts", [1, 2, 3, 16])
def test_split_program_every_point_as_alone(torch_dev, prec, npts):
    torch = torch_dev
    n = 5
    mom = torch.from_numpy(generate_events("gg_ttggg", n, first_event=3 * 10 ** 5)).cuda()
    p = split_handle(prec, npts, 0.0 if prec == "mixed" else None)
    w_in = torch.linspace(0.5, 2.0, n, dtype=torch.float64, device="cuda")
    me0 = torch.empty(n, dtype=torch.float64, device="cuda")
    out = p.reweight(mom, w_in=w_in, me_base_out=me0)
    base = p.eval_me(mom)
    ref = torch.stack([w_in * (p.eval_me(mom, point=k) / base) for k in range(npts)])
    if prec == "mixed":
        assert torch.equal(out, ref) and torch.equal(me0, base)
    else:
        assert (out / ref - 1).abs().max() <= FP64_TOL and (me0 / base - 1).abs().max() <= FP64_TOL


@pytest.mark.parametrize("prec,npts,n", [("mixed", 3, 340), ("mixed", 3, 1025), ("mixed", 16, 2100), ("fp64", 2, 70),
                                         ("fp64", 16, 1030)])
def test_split_program_batch_size_does_not_matter(torch_dev, prec, npts, n):
    """Single points and whole events per wave, one batch and several."""
    torch = torch_dev
    mom = torch.from_numpy(generate_events("gg_ttggg", n, first_event=10 ** 6)).cuda()
    p = split_handle(prec, npts)
    out = p.reweight(mom)
    for sel in (slice(0, 9), slice(n - 11, n)):
        assert torch.equal(out[:, sel], p.reweight(mom[:, :, sel].contiguous()))


def test_buffers_survive_handles_and_streams(torch_dev):
    """The library's memory pool: calls on two streams, handles created and
    destroyed between them, the same weights every time."""
    torch = torch_dev
    mom = torch.from_numpy(generate_events("gg_ttgg", 2000, first_event=5)).cuda()
    ref = handle("mixed", 4).reweight(mom)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    outs = []
    for i in range(6):
        p = handle("mixed", 4)
        with torch.cuda.stream(streams[i % 2]):
            outs.append(p.reweight(mom))
        if i % 3 == 2:
            torch.cuda.synchronize()
        p.close()
    torch.cuda.synchronize()
    assert all(torch.equal(o, ref) for o in outs)


# one event per lane and several events per wave sum the same helicity terms in
# another order, in double: NHEL rounding errors per |M|^2, three of those in a
# weight; in double precision the terms themselves are held to 1e-12
SUM_TOL = {"mixed": 3 * 32 * 2.0 ** -53, "fp64": FP64_TOL}


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("proc,n", [("gg_tt", 1), ("gg_tt", 15), ("gg_tt", 17), ("gg_tt", 106495), ("gg_tt", 126976),
                                    ("gg_ttg", 1), ("gg_ttg", 7), ("gg_ttg", 9), ("gg_ttg", 196607),
                                    ("gg_ttg", 196613)])
def test_several_events_per_wave(torch_dev, prec, proc, n):
    import paper_2312_07440_amd as mg
    torch = torch_dev
    mom = torch.from_numpy(generate_events(proc, min(n, 4099), first_event=11)).cuda()
    mom = mom.repeat(1, 1, -(-n // mom.shape[2]))[:, :, :n].contiguous()
    w_in = torch.linspace(0.5, 2.0, n, dtype=torch.float64, device="cuda")
    got, me = [], []
    for mapping in ("auto", "event_per_lane"):
        p = mg.Process(proc, prec)
        p.set_params([{"kappa_ttg": float(k), "alphas": 0.12} for k in kappa_points(3)])
        p.set_lane_mapping(mapping)
        got.append(p.reweight(mom, w_in=w_in))
        me.append(p.eval_me(mom, point=1))
    assert (got[0] / got[1] - 1).abs().max() <= SUM_TOL[prec]
    assert (me[0] / me[1] - 1).abs().max() <= SUM_TOL[prec]

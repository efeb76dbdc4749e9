"""The size of a batch selects the kernel.  Where the library cuts a call's
events into pieces itself, every piece takes the whole call's kernel:
mgrw_reweight_host states its results equal mgrw_reweight's bit for bit."""
import numpy as np
import pytest

from synth import generate_events, kappa_points

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def handle(proc, prec, npts=3):
    import paper_2312_07440_amd as mg
    p = mg.Process(proc, prec)
    p.set_params([{"kappa_ttg": float(k), "alphas": 0.118 * (1 + 0.01 * (i % 3))}
                  for i, k in enumerate(kappa_points(npts))])
    return p


def events(proc, n, distinct=4099):
    """n events [n_ext, 4, n], the first `distinct` of them repeated."""
    mom = generate_events(proc, min(n, distinct), first_event=11)
    return np.ascontiguousarray(np.tile(mom, (1, 1, -(-n // mom.shape[2])))[:, :, :n])


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("proc,n,chunk", [("gg_tt", (1 << 18) + 5, 0), ("gg_tt", 140001, 1000),
                                          ("gg_ttg", (1 << 18) + 5, 0), ("gg_ttg", 200003, 70000),
                                          ("gg_ttg", 131072, 65537), ("gg_tt", 65536, 30000)])
def test_host_chunks_equal_the_device_call(torch_dev, prec, proc, n, chunk):
    """Whole call, full chunks and last chunk on either side of the sizes that
    select the kernel."""
    torch = torch_dev
    mom = events(proc, n)
    w = np.random.default_rng(8).uniform(0.5, 2.0, n)
    p = handle(proc, prec)
    ref = p.reweight(torch.from_numpy(mom).cuda(), w_in=torch.from_numpy(w).cuda()).cpu().numpy()
    assert np.array_equal(p.reweight_host(mom, w_in=w, chunk=chunk), ref)


# both sides of each switch between the kernels and between their tiles, and a
# nearly empty and a full last round
SIZES = [("gg_tt", "mixed", 1, n) for n in (65535, 65536, 100000, 131072, 131073)]
SIZES += [("gg_tt", "fp64", npts, n) for npts in (1, 16) for n in (65536, 65537, 120000)]
SIZES += [("gg_ttg", prec, npts, n) for prec in ("mixed", "fp64") for npts in (1, 9) for n in (65536, 65537, 196609)]
# the helicity terms of an event are the same in both kernels, in double
# precision to 1e-12; their sums differ by at most NHEL roundings per |M|^2
SUM_TOL = {"mixed": 3 * 32 * 2.0 ** -53, "fp64": 2e-12}


@pytest.mark.parametrize("proc,prec,npts,n", SIZES)
def test_every_route_gives_the_same_weights(torch_dev, proc, prec, npts, n):
    torch = torch_dev
    mom = torch.from_numpy(events(proc, n)).cuda()
    w = torch.linspace(0.5, 2.0, n, dtype=torch.float64, device="cuda")
    p = handle(proc, prec, npts)
    out, me = p.reweight(mom, w_in=w), p.eval_me(mom, point=0)
    p.set_lane_mapping("event_per_lane")
    assert (out / p.reweight(mom, w_in=w) - 1).abs().max() <= SUM_TOL[prec]
    assert (me / p.eval_me(mom, point=0) - 1).abs().max() <= SUM_TOL[prec]


def test_more_events_than_one_launch_holds(torch_dev):
    """g g -> t tbar g, several threads per event: 2^29 events are 2^32 threads,
    which one launch does not take."""
    torch = torch_dev
    n = (1 << 29) + 33
    if torch.cuda.mem_get_info()[0] < 130 << 30:
        pytest.skip("needs 130 GiB of free device memory")
    base = torch.from_numpy(generate_events("gg_ttg", 4099, first_event=11)).cuda()
    p = handle("gg_ttg", "mixed", 2)   # three points in all: several events per wave
    me0_ref = torch.empty(4099, dtype=torch.float64, device="cuda")
    ref = p.reweight(base, me_base_out=me0_ref)
    reps = -(-n // 4099)
    mom = torch.empty(5, 4, n, dtype=torch.float64, device="cuda")
    for i in range(5):
        for mu in range(4):
            mom[i, mu] = base[i, mu].repeat(reps)[:n]
    out = torch.full((2, n), -1.0, dtype=torch.float64, device="cuda")
    me0 = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
    p.reweight(mom, out=out, me_base_out=me0)
    whole = n // 4099 * 4099
    for got, want in ((out[0], ref[0]), (out[1], ref[1]), (me0, me0_ref)):
        assert bool((got[:whole].view(-1, 4099) == want).all())
        assert torch.equal(got[whole:], want[: n - whole])
    del mom, out, me0
    torch.cuda.empty_cache()

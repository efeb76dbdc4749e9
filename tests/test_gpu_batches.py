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
                                          ("gg_ttg", (1 << 18) + 5, 0), ("gg_ttg", 200003, 70000)])
def test_host_chunks_equal_the_device_call(torch_dev, prec, proc, n, chunk):
    """Whole call, full chunks and last chunk on either side of the sizes that
    select the kernel."""
    torch = torch_dev
    mom = events(proc, n)
    w = np.random.default_rng(8).uniform(0.5, 2.0, n)
    p = handle(proc, prec)
    ref = p.reweight(torch.from_numpy(mom).cuda(), w_in=torch.from_numpy(w).cuda()).cpu().numpy()
    assert np.array_equal(p.reweight_host(mom, w_in=w, chunk=chunk), ref)


def test_more_events_than_one_launch_holds(torch_dev):
    """g g -> t tbar g, several threads per event: 2^29 events are 2^32 threads,
    which one launch does not take."""
    torch = torch_dev
    n = (1 << 29) + 33
    if torch.cuda.mem_get_info()[0] < 130 << 30:
        pytest.skip("needs 130 GiB of free device memory")
    base = torch.from_numpy(generate_events("gg_ttg", 4099, first_event=11)).cuda()
    p = handle("gg_ttg", "mixed")
    ref = p.eval_me(base)
    reps = -(-n // 4099)
    mom = torch.empty(5, 4, n, dtype=torch.float64, device="cuda")
    for i in range(5):
        for mu in range(4):
            mom[i, mu] = base[i, mu].repeat(reps)[:n]
    out = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
    p.eval_me(mom, out=out)
    whole = n // 4099 * 4099
    assert bool((out[:whole].view(-1, 4099) == ref).all())
    assert torch.equal(out[whole:], ref[: n - whole])
    del mom, out
    torch.cuda.empty_cache()

"""Input weights in the place of an output: w_in may be a row of w_out or
me_base_out itself, for every process and exact call, also where events are
evaluated a second time in double precision (that pass reads the weights
again) and in every chunk of the allocation-free call."""
import pytest

from synth import alpha_points, generate_events, kappa_points

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def handle(proc, prec, tau):
    import paper_2312_07440_amd as mg
    p = mg.Process(proc, prec, {"alpha": 1 / 132.5} if proc == "ee_5a" else None)
    if proc == "ee_mumu":
        p.set_params([{"mz": 95.0}, {"mz": 90.0}])
    elif proc == "ee_5a":
        p.set_params([{"alpha": float(a)} for a in alpha_points(2)])
    else:
        p.set_params([{"kappa_ttg": float(k)} for k in kappa_points(2)])
    if tau is not None:
        p.set_rescue_threshold(tau)
    return p


CASES = [(proc, prec, None, call)
         for proc, prec in (("ee_mumu", "fp64"), ("gg_tt", "mixed"), ("gg_ttgg", "fp64"), ("ee_5a", "mixed"))
         for call in ("reweight", "reweight_noalloc", "reweight_kpoly") if (proc, call) != ("ee_mumu", "reweight_kpoly")]
# with re-evaluated events: a few of them, and all
CASES += [(proc, "mixed", tau, call) for proc in ("gg_ttg", "gg_ttgg") for tau in (0.05, 1.0)
          for call in ("reweight", "reweight_noalloc", "reweight_kpoly")]
CASES += [("gg_ttggg", "mixed", 0.05, "reweight"), ("gg_ttggg", "fp64", None, "reweight")]


@pytest.mark.parametrize("proc,prec,tau,call", CASES)
def test_weights_in_place(torch_dev, proc, prec, tau, call):
    torch = torch_dev
    n = 40 if proc == "gg_ttggg" else 3001
    mom = torch.from_numpy(generate_events(proc, n, first_event=77)).cuda()
    p = handle(proc, prec, tau)
    w = torch.linspace(0.5, 2.0, n, dtype=torch.float64, device="cuda")
    me_ref = torch.empty(n, dtype=torch.float64, device="cuda")
    ref = getattr(p, call)(mom, w_in=w, me_base_out=me_ref)
    for place in (0, 1, "me"):
        buf = torch.zeros(2, n, dtype=torch.float64, device="cuda")
        me = torch.zeros(n, dtype=torch.float64, device="cuda")
        w_in = me if place == "me" else buf[place]
        w_in.copy_(w)
        getattr(p, call)(mom, w_in=w_in, out=buf, me_base_out=me)
        assert torch.equal(buf, ref) and torch.equal(me, me_ref), place


def test_weights_in_place_chunks(torch_dev):
    """More events than a chunk of the allocation-free call holds when it sets
    the weights aside (16777168 of g g -> t tbar g)."""
    torch = torch_dev
    n, m = 16777168 + 1001, 4099
    base = torch.from_numpy(generate_events("gg_ttg", m, first_event=77)).cuda()
    mom = base.repeat(1, 1, -(-n // m))[:, :, :n].contiguous()
    p = handle("gg_ttg", "mixed", 0.05)
    w = torch.linspace(0.5, 2.0, n, dtype=torch.float64, device="cuda")
    ref = p.reweight(mom, w_in=w)
    buf = torch.zeros(2, n, dtype=torch.float64, device="cuda")
    buf[1] = w
    p.reweight_noalloc(mom, w_in=buf[1], out=buf)
    assert torch.equal(buf, ref)

"""The FP64 kernels of the colour-ordered recursion at the edges of their 64-event blocks, through
every call that reads their colour-flow amplitudes: the fused colour sum, the separate one, the
per-helicity values and the colour-flow draws; and with massless tops, where a workgroup's four
quark spin configurations are not all good helicities.  The bar is the repository's FP64 bar:
1e-12 per event against the oracle, with the long-double referee beyond it."""
import numpy as np
import pytest
import torch

import oracle
from tests import referee
from tests import workloads as W

pytestmark = pytest.mark.gpu

PROCESSES = ["ee_mumu", "gg_tt", "gg_ttg", "gg_ttgg", "gg_ttggg"]


def check(name, p, got, params):
    want = oracle.me_batch(name, p, params=params)
    for i in np.where(~(np.abs(got / want - 1) <= referee.TOL))[0]:
        ok, r, spread = referee.judge(name, p[i], got[i], params)
        assert ok, (name, int(i), r, spread)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129])
@pytest.mark.parametrize("name", PROCESSES)
def test_block_edges(name, n):
    from paper_2210_11122_amd import Process
    # the largest case also crosses the batch size from which the process takes another kernel
    last = {"ee_mumu": 65665, "gg_tt": 65665, "gg_ttg": 16385, "gg_ttgg": 129, "gg_ttggg": 65}
    n = last[name] if n == 129 else n
    print(f"case recursion {name} n={n}", flush=True)
    proc = Process(name, m_top=W.M_TOP, alpha_em=W.ALPHA_EM, alpha_s=W.ALPHA_S)
    p = oracle.rambo(31, W.sqrt_s(name), W.final_masses(name), n)
    x = torch.from_numpy(p).cuda()
    me = proc.sigma(x)
    check(name, p, me.cpu().numpy(), W.PARAMS)
    tot, hel = proc.sigma(x, per_helicity=True)
    assert torch.equal(tot, me)
    assert np.allclose(hel.cpu().numpy().sum(axis=1) / proc.info["avg_factor"], me.cpu().numpy(), rtol=1e-13, atol=0)
    # uniforms at both ends of [0, 1): the draws end at the first and last flow of positive weight
    zero, one = torch.zeros(n, dtype=torch.float64).cuda(), torch.full((n,), 1 - 2.0 ** -53, dtype=torch.float64).cuda()
    sel, h0, c0 = proc.select(x, zero, zero)
    _, h1, c1 = proc.select(x, one, one)
    assert torch.equal(sel, me) and bool((c0 == 0).all()) and bool((c1 == proc.info["n_colors"] - 1).all())
    # the same events through the separate colour sum
    proc.set_fused_colour(False)
    assert torch.equal(proc.sigma(x), me)
    good = proc.good_helicities_index()
    assert bool((h0 == good[0]).all()) and bool((h1 == good[-1]).all())


@pytest.mark.parametrize("n", [65, 4161, 16385])
def test_channel_weights_in_the_kernel(n):
    """gg_tt and gg_ttg form the channel weights in the recursion kernels (gg_ttg with one spin configuration
    per lane up to 4096 events, four above): they sum to one over the channels, the mixed forms' diagram
    program gives the same weights to its own precision (1e-5), and without a channel |M|^2 is sigma's"""
    from paper_2210_11122_amd import Process
    for name in ("gg_tt", "gg_ttg"):
        print(f"case channels {name} n={n}", flush=True)
        a = dict(m_top=W.M_TOP, alpha_em=W.ALPHA_EM, alpha_s=W.ALPHA_S)
        proc, mixed = Process(name, **a), Process(name, precision="mixed_fp16", **a)
        x = torch.from_numpy(oracle.rambo(35, W.sqrt_s(name), W.final_masses(name), n)).cuda()
        me, me32 = proc.sigma(x), mixed.sigma(x)
        total = torch.zeros_like(me)
        for c in range(proc.info["n_diagrams"]):
            ch = torch.full((n,), c, dtype=torch.int32, device="cuda")
            got = proc.sigma_channel(x, ch)
            total += got
            assert torch.allclose(got / me, mixed.sigma_channel(x, ch) / me32, rtol=1e-3, atol=1e-5)
        assert torch.allclose(total, me, rtol=1e-13, atol=0)
        assert torch.equal(proc.sigma_channel(x, torch.full((n,), -1, dtype=torch.int32, device="cuda")), me)


@pytest.mark.parametrize("name,n", [("gg_tt", 65), ("gg_ttg", 65), ("gg_ttgg", 65), ("gg_ttggg", 3)])
def test_massless_tops_leave_spin_configurations_out(name, n):
    from paper_2210_11122_amd import Process
    print(f"case recursion massless {name} n={n}", flush=True)
    params = (0.0, W.ALPHA_EM, W.ALPHA_S)
    proc = Process(name, m_top=0.0, alpha_em=W.ALPHA_EM, alpha_s=W.ALPHA_S)
    spins = {}
    for lam in proc.good_helicities():
        spins.setdefault(lam[:2] + lam[4:], set()).add(lam[2:4])
    assert all(len(s) < 4 for s in spins.values())
    p = oracle.rambo(33, W.sqrt_s(name), [0.0] * (W.n_par(name) - 2), n)
    check(name, p, proc.sigma(torch.from_numpy(p).cuda()).cpu().numpy(), params)


@pytest.mark.parametrize("name,n", [("gg_ttg", 65), ("gg_ttg", 4161), ("gg_ttgg", 1), ("gg_ttgg", 1000)])
def test_rows_and_flow_weights_from_the_kernel(name, n):
    """the per-helicity output and the draws from the values that the amplitude kernel writes, against those
    from the jamps in memory (the separate colour sum): |M_h|^2 bitwise, and the draws the same (their weights
    differ by the order of a sum, 1e-15, so a uniform would have to lie that close to a boundary)"""
    from paper_2210_11122_amd import Process
    proc = Process(name, m_top=W.M_TOP, alpha_em=W.ALPHA_EM, alpha_s=W.ALPHA_S)
    x = proc.rambo(7, W.sqrt_s(name), n)
    g = torch.Generator(device="cuda").manual_seed(5)
    u = torch.rand((2, n), generator=g, dtype=torch.float64, device="cuda")
    got = [(*proc.sigma(x, per_helicity=True), *proc.select(x, u[0].contiguous(), u[1].contiguous()))]
    proc.set_fused_colour(False)
    got.append((*proc.sigma(x, per_helicity=True), *proc.select(x, u[0].contiguous(), u[1].contiguous())))
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_near_beam_events_keep_their_values():
    """Events with a gluon along a beam, whose P^2 = (k - k')^2 has lost half its digits, so that |M|^2 follows the
    rounding of P^2: the values are those of the diagram program (Cartesian P^2).  Bar 1e-11, ten times the FP64 bar,
    for what the two programs round differently; P^2 rounded in another way moves them by 2e-9 to 6e-8.  And they
    are within the event's conditioning of the long-double value."""
    import json
    import os
    from paper_2210_11122_amd import Process
    with open(os.path.join(os.path.dirname(__file__), "golden", "near_beam_events.json")) as fh:
        events = json.load(fh)["events"]
    for i, ev in enumerate(events):
        name = ev["process"]
        print(f"case near beam {name} {i}", flush=True)
        p = np.array([[float.fromhex(v) for v in row] for row in ev["momenta"]])
        want = float.fromhex(ev["me2"])
        proc = Process(name, m_top=W.M_TOP, alpha_em=W.ALPHA_EM, alpha_s=W.ALPHA_S)
        for n in (1, 5000 if name == "gg_ttg" else 70):   # gg_ttg: either of its kernels
            x = torch.from_numpy(np.broadcast_to(p, (n, *p.shape)).copy()).cuda()
            got = proc.sigma(x).cpu().numpy()
            assert np.all(np.abs(got / want - 1) < 1e-11), (name, i, n, np.abs(got / want - 1).max())
        ok, rel, spread = referee.judge(name, p, got[0], W.PARAMS)
        assert ok, (name, i, rel, spread)


@pytest.mark.parametrize("name,n", [("ee_mumu", 257), ("gg_tt", 1), ("gg_tt", 4161), ("gg_ttg", 4096), ("gg_ttg", 4161)])
def test_channel_weights_do_not_depend_on_the_route(name, n):
    """The channel weights of a batch, of slices of it and with the separate colour sum: the same bits, with every
    diagram's id among the events, none (-1) and one past the last."""
    from paper_2210_11122_amd import Process
    print(f"case channel routes {name} n={n}", flush=True)
    proc = Process(name, m_top=W.M_TOP, alpha_em=W.ALPHA_EM, alpha_s=W.ALPHA_S)
    x = proc.rambo(9, W.sqrt_s(name), n)
    nd = proc.info["n_diagrams"]
    ch = (torch.arange(n, device="cuda") % (nd + 2) - 1).to(torch.int32)
    whole = proc.sigma_channel(x, ch)
    slices = [proc.sigma_channel(x[i:i + 1387].contiguous(), ch[i:i + 1387].contiguous()) for i in range(0, n, 1387)]
    assert torch.isfinite(whole).all() and bool((whole[ch >= nd] == 0).all())
    assert torch.equal(torch.cat(slices), whole)
    proc.set_fused_colour(False)
    assert torch.equal(proc.sigma_channel(x, ch), whole)


@pytest.mark.parametrize("name,m_top,n", [("gg_ttg", 0.0, 65), ("gg_ttgg", 0.0, 65), ("gg_ttgg", W.M_TOP, 0)])
def test_rows_and_flow_weights_massless_and_over_chunks(name, m_top, n):
    """as test_rows_and_flow_weights_from_the_kernel, with massless tops, where some quark spins have no row and must
    neither store one nor add to the flow weights, and (n = 0) for a batch of one chunk and a ragged one"""
    from paper_2210_11122_amd import Process
    proc = Process(name, m_top=m_top, alpha_em=W.ALPHA_EM, alpha_s=W.ALPHA_S)
    n = n or proc.info["chunk_events"] + 37
    print(f"case rows {name} m_top={m_top} n={n}", flush=True)
    x = proc.rambo(8, W.sqrt_s(name), n)
    u = torch.rand((2, n), generator=torch.Generator(device="cuda").manual_seed(6), dtype=torch.float64, device="cuda")
    got = []
    for fused in (True, False):
        proc.set_fused_colour(fused)
        got.append((proc.sigma(x), *proc.sigma(x, per_helicity=True), *proc.select(x, u[0].contiguous(), u[1].contiguous())))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    assert torch.equal(got[0][0], got[0][1]) and torch.equal(got[0][0], got[0][3])

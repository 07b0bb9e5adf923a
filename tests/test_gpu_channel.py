"""GPU single-diagram channel weights (me_sigma_channel) against the oracle's own Feynman
diagrams (oracle/diagrams.py: enumeration, Lorentz parts and colour factors of its own).
Diagrams are matched by their internal lines, so the two numberings need not agree."""
import numpy as np
import pytest
import torch

import oracle
from oracle import diagrams as Dg
from tests import workloads as W

pytestmark = pytest.mark.gpu


def make_process(name, precision="fp64"):
    from paper_2210_11122_amd import Process
    return Process(name, m_top=W.M_TOP, alpha_em=W.ALPHA_EM, alpha_s=W.ALPHA_S, precision=precision)


@pytest.mark.parametrize("name,n_evt,n_chan", [("gg_tt", 4, 3), ("gg_ttg", 3, 16), ("gg_ttgg", 2, 12)])
def test_channel_weights_match_oracle(name, n_evt, n_chan):
    print(f"case channel weights {name}", flush=True)
    proc = make_process(name)
    lines = proc.diagrams()
    assert len(lines) == proc.info["n_diagrams"]
    ng = oracle.n_par(name) - 2
    assert set(lines) == {Dg.descriptor(name, d) for d in Dg.diagrams(ng)}
    p = oracle.rambo(41, W.sqrt_s(name), W.final_masses(name), n_evt)
    chans = np.linspace(0, len(lines) - 1, n_chan).astype(np.int32)
    x = torch.from_numpy(np.repeat(p, len(chans), axis=0)).cuda()
    ch = torch.from_numpy(np.tile(chans, n_evt)).cuda()
    got = proc.sigma_channel(x, ch).cpu().numpy().reshape(n_evt, len(chans))
    me = proc.sigma(torch.from_numpy(p).cuda()).cpu().numpy()
    K = Dg.colour_weights_K(name)
    # the oracle's own helicity filter (same recipe as the library's pre-pass)
    good = oracle.good_helicities(name, W.sqrt_s(name), W.final_masses(name), W.PARAMS)
    assert sorted(proc.good_helicities_index()) == good
    for e in range(n_evt):
        Wd = Dg.diagram_weights(name, p[e], W.PARAMS, K, helicities=good)
        tot = sum(Wd.values())
        for k, c in enumerate(chans):
            want = me[e] * Wd[lines[c]] / tot
            assert got[e, k] == pytest.approx(want, rel=1e-12), (e, int(c))


def test_channel_weights_ttggg_match_oracle():
    """gg_ttggg: the weights of 24 channels of two events against the oracle's W_d.  The
    oracle's colour weights K_ds and its helicity filter take about a minute, so they come
    from tests/golden/gg_ttggg_channel_tables.json (written by the script beside it, which
    calls only the oracle); a sample of K_ds is recomputed here."""
    import json
    import os
    name = "gg_ttggg"
    print(f"case channel weights {name} vs oracle", flush=True)
    tab = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "gg_ttggg_channel_tables.json")))
    ents = Dg.entries(name)
    assert [tuple(e["lines"]) for e in tab["entries"]] == [Dg.descriptor(name, d) for d, _ in ents]
    assert [tuple(e["assign"]) for e in tab["entries"]] == [tuple(s) for _, s in ents]
    K = np.array([e["K"] for e in tab["entries"]])
    for i in range(0, len(ents), 97):
        d, s = ents[i]
        assert np.sum(np.abs(Dg.colour_tensor(d, s, 5)) ** 2) == pytest.approx(K[i], rel=1e-13)
    good = tab["good_helicities"]
    proc = make_process(name)
    lines = proc.diagrams()
    assert set(lines) == {Dg.descriptor(name, d) for d, _ in ents}
    assert sorted(proc.good_helicities_index()) == good
    p = oracle.rambo(45, W.sqrt_s(name), W.final_masses(name), 2)
    me = proc.sigma(torch.from_numpy(p).cuda()).cpu().numpy()
    for e in range(2):
        Wd = Dg.diagram_weights(name, p[e], W.PARAMS, K, helicities=good)
        tot = sum(Wd.values())
        # spread over the numbering, plus the event's three largest channels
        top = sorted(range(len(lines)), key=lambda c: -Wd[lines[c]])[:3]
        chans = np.array(sorted(set(np.linspace(0, len(lines) - 1, 21).astype(int)) | set(top)), dtype=np.int32)
        x = torch.from_numpy(np.repeat(p[e:e + 1], len(chans), axis=0)).cuda()
        got = proc.sigma_channel(x, torch.from_numpy(chans).cuda()).cpu().numpy()
        for k, c in enumerate(chans):
            want = me[e] * Wd[lines[c]] / tot
            assert got[k] == pytest.approx(want, rel=1e-12), (e, int(c))


def test_channel_weights_sum_to_one_and_no_channel():
    name = "gg_ttgg"
    proc = make_process(name)
    nd = proc.info["n_diagrams"]
    p = oracle.rambo(42, W.sqrt_s(name), W.final_masses(name), 3)
    x = torch.from_numpy(np.repeat(p, nd, axis=0)).cuda()
    ch = torch.from_numpy(np.tile(np.arange(nd, dtype=np.int32), 3)).cuda()
    got = proc.sigma_channel(x, ch).cpu().numpy().reshape(3, nd)
    me = proc.sigma(torch.from_numpy(p).cuda()).cpu().numpy()
    assert np.all(got >= 0)
    assert np.allclose(got.sum(axis=1), me, rtol=1e-12)
    none = proc.sigma_channel(torch.from_numpy(p).cuda(), torch.full((3,), -1, dtype=torch.int32).cuda())
    assert np.array_equal(none.cpu().numpy(), me)


@pytest.mark.parametrize("precision", ["fp64", "mixed_fp16"])
def test_channel_weights_ttggg(precision):
    """gg_ttggg (segment kernels add their sums in turn): the weights of all 1240 channels
    of an event sum to one"""
    print(f"case channel weights gg_ttggg {precision}", flush=True)
    name = "gg_ttggg"
    proc = make_process(name, precision)
    nd = proc.info["n_diagrams"]
    assert nd == 1240
    p = oracle.rambo(43, W.sqrt_s(name), W.final_masses(name), 2)
    x = torch.from_numpy(np.repeat(p, nd, axis=0)).cuda()
    ch = torch.from_numpy(np.tile(np.arange(nd, dtype=np.int32), 2)).cuda()
    got = proc.sigma_channel(x, ch).cpu().numpy().reshape(2, nd)
    me = proc.sigma(torch.from_numpy(p).cuda()).cpu().numpy()
    tol = 1e-12 if precision == "fp64" else 1e-5
    assert np.all(got >= 0) and np.allclose(got.sum(axis=1), me, rtol=tol)


def test_channel_rejects():
    import ctypes
    from paper_2210_11122_amd import binding
    L = binding.load()
    gg = make_process("gg_gg")
    x = torch.zeros((4, 4, 4), dtype=torch.float64, device="cuda")
    out = torch.empty(4, dtype=torch.float64, device="cuda")
    ch = torch.zeros(4, dtype=torch.int32, device="cuda")
    v = lambda t: ctypes.c_void_p(t.data_ptr())
    assert L.me_sigma_channel(gg._h, v(x), 4, v(ch), v(out), None) == -1
    tt = make_process("gg_tt")
    host = np.zeros(4, dtype=np.int32)
    assert L.me_sigma_channel(tt._h, v(x), 4, ctypes.c_void_p(host.ctypes.data), v(out), None) == -1


def test_channel_weights_ee_mumu_z():
    """photon (diagram 0) and Z (diagram 1): W_d = sum_h |A_d|^2 from the oracle's amplitudes
    of each diagram alone"""
    name = "ee_mumu_z"
    proc = make_process(name)
    assert proc.info["n_diagrams"] == 2
    for rs in (500.0, 91.188):
        p = oracle.rambo(44, rs, [0.0, 0.0], 8)
        x = torch.from_numpy(np.repeat(p, 2, axis=0)).cuda()
        ch = torch.from_numpy(np.tile(np.array([0, 1], dtype=np.int32), 8)).cuda()
        got = proc.sigma_channel(x, ch).cpu().numpy().reshape(8, 2)
        me = proc.sigma(torch.from_numpy(p).cuda()).cpu().numpy()
        for e in range(8):
            wg = sum(abs(oracle.ee_z_amplitude(p[e], h, 1, W.PARAMS)) ** 2 for h in range(16))
            wz = sum(abs(oracle.ee_z_amplitude(p[e], h, 2, W.PARAMS)) ** 2 for h in range(16))
            assert got[e, 0] == pytest.approx(me[e] * wg / (wg + wz), rel=1e-12)
            assert got[e, 1] == pytest.approx(me[e] * wz / (wg + wz), rel=1e-12)


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("name", ["gg_tt", "gg_ttg"])
def test_channel_weights_of_a_large_batch_match_oracle(name, fused):
    """every channel of three events, repeated to 4161: gg_ttg then takes the kernel that sums the helicities and
    applies the weight itself or, with the separate colour sum, the one with all spins in a lane"""
    print(f"case channel weights {name} large batch, fused={fused}", flush=True)
    proc = make_process(name)
    proc.set_fused_colour(fused)
    lines = proc.diagrams()
    p = oracle.rambo(41, W.sqrt_s(name), W.final_masses(name), 3)
    i = np.arange(4161)
    ev, ch = i % 3, (i // 3 % len(lines)).astype(np.int32)
    got = proc.sigma_channel(torch.from_numpy(p[ev]).cuda(), torch.from_numpy(ch).cuda()).cpu().numpy()
    me = proc.sigma(torch.from_numpy(p).cuda()).cpu().numpy()
    K = Dg.colour_weights_K(name)
    good = oracle.good_helicities(name, W.sqrt_s(name), W.final_masses(name), W.PARAMS)
    want = np.empty((3, len(lines)))
    for e in range(3):
        Wd = Dg.diagram_weights(name, p[e], W.PARAMS, K, helicities=good)
        want[e] = [me[e] * Wd[l] / sum(Wd.values()) for l in lines]
    assert np.all(np.abs(got / want[ev, ch] - 1) < 1e-12)

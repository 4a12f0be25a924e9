"""GPU blending, pseudo-deblending, re-sorting and survey-level separation
against the FP64 oracle (oracle/blending.py, oracle.robust_invert per
receiver gather), through the C ABI."""
import numpy as np
import pytest

import oracle
from oracle import blending as OB
from oracle.irls import IrlsParams
from synth import make_survey
from tests.gpu_common import rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import torch
    import paper_1711_10214_amd as A
    assert torch.cuda.is_available()
    return A


def test_blend_deblend_resort_match_oracle(A):
    import torch
    from paper_1711_10214_amd import survey as S
    sv = make_survey(ns=12, nt=128, seed=3)
    D = torch.tensor(sv.D, dtype=torch.float32, device="cuda")
    b = S.blend(D, sv.fire)
    Df = sv.D.astype(np.float32).astype(np.float64)
    b_ref = OB.blend(Df, sv.fire)
    assert rel_l2(b.cpu().numpy(), b_ref) <= 1e-6
    c_ref = OB.deblend(b_ref, sv.fire, 128)
    bt = torch.tensor(b_ref, dtype=torch.float32, device="cuda")
    c_src = S.deblend(bt, sv.fire, 12, 128, receiver_major=False).cpu().numpy()
    c_rcv = S.deblend(bt, sv.fire, 12, 128, receiver_major=True).cpu().numpy()
    assert rel_l2(c_src, c_ref) <= 1e-7
    assert np.array_equal(c_rcv, np.transpose(c_src, (1, 0, 2)))
    assert np.array_equal(S.resort(torch.tensor(c_src, device="cuda")).cpu().numpy(), c_rcv)


def test_survey_separation_matches_oracle(A):
    """16 sources x 16 receivers: every receiver gather separated in one
    batched solve equals the oracle's per-gather solve."""
    import torch
    from paper_1711_10214_amd import survey as S
    sv = make_survey(ns=16, nt=256, seed=4, n_events=4)
    vel = list(np.linspace(1500.0, 3200.0, 6))
    D = torch.tensor(sv.D, dtype=torch.float32, device="cuda")
    b = S.blend(D, sv.fire)
    prm = A.Params(p=1, q=2, n_outer=3, n_inner=5)
    print("[gpu] survey separation 16 x 16 x 256", flush=True)
    csg = S.separate(b, sv.fire, 16, 256, sv.dt, sv.dx, vel, prm, fmax=100.0).cpu().numpy()
    b_np = b.cpu().numpy().astype(np.float64)
    crg = np.transpose(OB.deblend(b_np, sv.fire, 256), (1, 0, 2))
    g = oracle.geometry(256, 16, sv.dt, sv.dx, vel, fmax=100.0)
    sep = np.stack([oracle.robust_invert(g, crg[r], IrlsParams(p=1, q=2, n_outer=3, n_inner=5))[1]
                    for r in range(16)])
    csg_ref = np.transpose(sep, (1, 0, 2))
    e = rel_l2(csg, csg_ref)
    q_sep = oracle.q_db(sv.D, csg)
    q_pd = oracle.q_db(sv.D, np.transpose(crg, (1, 0, 2)))
    print(f"  rel-L2 vs oracle {e:.2e}; Q separated {q_sep:.2f} dB, pseudo-deblended {q_pd:.2f} dB", flush=True)
    assert e <= 1e-4
    assert q_sep > q_pd


# Edges of the kernels' tiles: 1 or 4 samples per thread, 256 or 1024 record
# samples per workgroup, 512 sources tested at a time; shots that start together,
# out of order, and past the record.
SURVEY_EDGES = [(1, 1, 1, 1), (3, 2, 3, 5), (5, 9, 7, 40), (4, 8, 1024, 1023), (6, 3, 130, 1025), (1030, 2, 5, 2051)]
# Many shots over every sample, one and four samples per thread.
SURVEY_EDGES += [(70, 3, 33, 40), (515, 5, 300, 700), (40, 600, 300, 2048), (3, 1000, 5, 1000)]
# Several receivers per workgroup (a 1024th of receivers x record tiles, at most
# 8), the last workgroup short: 2, 3, 4 and 8; 4 with three lists of sources.
SURVEY_EDGES += [(2, 2049, 6, 900), (4, 1601, 9, 1100), (3, 2051, 7, 1025), (2, 4099, 5, 1030), (1025, 2050, 2, 1026)]


@pytest.mark.parametrize("ns,nr,nt,nrec", SURVEY_EDGES)
def test_survey_tile_edges(A, ns, nr, nt, nrec):
    """Blending adds the shots in index order in FP32, so it equals numpy's
    running FP32 sum; pseudo-deblending and re-sorting copy."""
    import torch
    from paper_1711_10214_amd import survey as S
    print(f"[gpu] survey edges {ns} x {nr} x {nt}, {nrec} record samples", flush=True)
    rng = np.random.default_rng(ns + nt)
    D = rng.standard_normal((ns, nr, nt)).astype(np.float32)
    fire = rng.integers(0, max(1, nrec), ns).astype(np.int32)
    fire[::7] = fire[0]
    b = np.zeros((nr, nrec), np.float32)
    for s in range(ns):
        n = min(nt, nrec - int(fire[s]))
        b[:, fire[s]:fire[s] + n] += D[s, :, :n]
    g = S.blend(torch.tensor(D, device="cuda"), fire, nrec)
    assert np.array_equal(g.cpu().numpy(), b)
    pad = np.concatenate([b, np.zeros((nr, nt), np.float32)], axis=1)
    c = np.stack([pad[:, f:f + nt] for f in fire])
    assert np.array_equal(S.deblend(g, fire, ns, nt, receiver_major=False).cpu().numpy(), c)
    r = S.deblend(g, fire, ns, nt)
    assert np.array_equal(r.cpu().numpy(), np.transpose(c, (1, 0, 2)))
    assert np.array_equal(S.resort(r).cpu().numpy(), c)

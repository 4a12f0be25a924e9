"""GPU time-domain (classical) ASHRT / AASHRT pair against the brute-force
FP64 time-domain reference (oracle/timedomain.py), through the C ABI
(ashrt_td_forward, ashrt_td_adjoint).  Bar: relative L2 <= 1e-5 (FP64 curve
times, FP32 sums) and the FP32 dot-product test."""
import numpy as np
import pytest

from oracle import timedomain as TD
from tests.gpu_common import f32, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import torch
    import paper_1711_10214_amd as A
    assert torch.cuda.is_available()
    return A


CASES = {
    "ashrt-3v": dict(nt=96, nx=24, dt=0.004, dx=12.5, vel=[1500.0, 2200.0, 3400.0], tau0=None),
    "aashrt-ragged": dict(nt=77, nx=19, dt=0.004, dx=10.0, vel=[1800.0, 1800.0, 2600.0, 2600.0], tau0=[0, 6, 0, 11]),
    "zero-velocity": dict(nt=64, nx=16, dt=0.004, dx=12.5, vel=[0.0, 2000.0], tau0=None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_time_domain_pair_matches_reference(A, name):
    import torch
    c = CASES[name]
    print(f"[gpu] time-domain pair case={name}", flush=True)
    rng = np.random.default_rng(5)
    P = len(c["vel"])
    m = f32(rng.standard_normal((P, c["nx"], c["nt"])))
    d = f32(rng.standard_normal((c["nx"], c["nt"])))
    plan = A.Plan(c["nt"], c["nx"], c["dt"], c["dx"], c["vel"], tau0=c["tau0"])
    mt = torch.tensor(m, dtype=torch.float32, device="cuda")
    dt_ = torch.tensor(d, dtype=torch.float32, device="cuda")
    fg = plan.td_forward(mt).cpu().numpy()
    ag = plan.td_adjoint(dt_).cpu().numpy()
    vel = np.asarray(c["vel"], float)
    tau0 = np.zeros(P, int) if c["tau0"] is None else np.asarray(c["tau0"])
    live = vel > 0
    fr = TD.forward(m[live], c["dt"], c["dx"], vel[live], tau0[live])
    ar = np.zeros_like(m)
    ar[live] = TD.adjoint(d, c["dt"], c["dx"], vel[live], tau0[live])
    # v = 0: the curve collapses onto its apex trace, t = tau0 + tau
    for p in np.flatnonzero(~live):
        n0 = int(tau0[p])
        fr[:, n0:] += m[p][:, :c["nt"] - n0]
        ar[p][:, :c["nt"] - n0] = d[:, n0:]
    ef, ea = rel_l2(fg, fr), rel_l2(ag, ar)
    print(f"  forward {ef:.2e} adjoint {ea:.2e}", flush=True)
    assert ef <= 1e-5 and ea <= 1e-5
    lhs = float(np.sum(fg.astype(np.float64) * d))
    rhs = float(np.sum(m * ag.astype(np.float64)))
    assert abs(lhs - rhs) <= 1e-5 * np.linalg.norm(fg) * np.linalg.norm(d)


def test_time_domain_mask(A):
    import torch
    rng = np.random.default_rng(6)
    nt, nx, vel = 80, 20, [1700.0, 2900.0]
    mask = (rng.uniform(size=nx) > 0.4).astype(np.uint8)
    m = f32(rng.standard_normal((2, nx, nt)))
    d = f32(rng.standard_normal((nx, nt)))
    plan = A.Plan(nt, nx, 0.004, 12.5, vel)
    mk = torch.tensor(mask, device="cuda")
    fg = plan.td_forward(torch.tensor(m, dtype=torch.float32, device="cuda"), mask=mk).cpu().numpy()
    ag = plan.td_adjoint(torch.tensor(d, dtype=torch.float32, device="cuda"), mask=mk).cpu().numpy()
    fr = TD.forward(m, 0.004, 12.5, vel) * mask[:, None]
    ar = TD.adjoint(d * mask[:, None], 0.004, 12.5, vel)
    assert rel_l2(fg, fr) <= 1e-5 and rel_l2(ag, ar) <= 1e-5


# Edges of the kernels' tiles (64 times, 8 traces, windows of 4 samples) and of
# the record: shortest traces, shifts past the record, curves that leave it,
# flat apexes (a far trace at a low velocity spans many apex times per sample).
EDGES = [
    (2, 2, [2000.0], [0]), (3, 5, [1500.0, 0.0], [1, 0]), (4, 8, [900.0], [0]), (5, 9, [3000.0], [2]),
    (63, 7, [1500.0, 2500.0], [0, 70]), (64, 8, [400.0], [0]), (65, 17, [1500.0], [64]), (130, 33, [600.0, 5000.0], [3, 0]),
]


@pytest.mark.parametrize("nt,nx,vel,tau0", EDGES)
def test_time_domain_tile_edges(A, nt, nx, vel, tau0):
    """Same bar as above; dead traces hold NaN, which must not reach any output."""
    import torch
    print(f"[gpu] time-domain edges {nt} x {nx}", flush=True)
    rng = np.random.default_rng(nt)
    P = len(vel)
    m = f32(rng.standard_normal((P, nx, nt)))
    d = f32(rng.standard_normal((nx, nt)))
    mask = np.ones(nx, np.uint8)
    mask[1::3] = 0
    plan = A.Plan(nt, nx, 0.004, 12.5, vel, tau0=tau0, ntp=max(8, 1 << (2 * nt - 1).bit_length()),
                  nxp=max(4, 1 << (2 * nx - 1).bit_length()))
    dn = np.where(mask[:, None] == 0, np.nan, d)
    mk = torch.tensor(mask, device="cuda")
    fg = plan.td_forward(torch.tensor(m, dtype=torch.float32, device="cuda"), mask=mk).cpu().numpy()
    ag = plan.td_adjoint(torch.tensor(dn, dtype=torch.float32, device="cuda"), mask=mk).cpu().numpy()
    fr, ar = np.zeros((nx, nt)), np.zeros_like(m)
    d0 = d * mask[:, None]
    for p, (v, n0) in enumerate(zip(vel, tau0)):
        if v > 0:
            fr += TD.forward(m[p:p + 1], 0.004, 12.5, [v], [n0])
            ar[p] = TD.adjoint(d0, 0.004, 12.5, [v], [n0])[0]
        elif n0 < nt:
            fr[:, n0:] += m[p][:, :nt - n0]
            ar[p][:, :nt - n0] = d0[:, n0:]
    fr *= mask[:, None]
    assert np.isfinite(fg).all() and np.isfinite(ag).all()
    assert np.linalg.norm(fg - fr) <= 1e-5 * max(np.linalg.norm(fr), 1e-3)
    assert np.linalg.norm(ag - ar) <= 1e-5 * max(np.linalg.norm(ar), 1e-3)


# Impulses (apex trace, apex time) per velocity and shift: steep and flat parts
# of the curves, the apex itself, weights near 0 and 1.
@pytest.mark.parametrize("v,n0", [(1500.0, 0), (2345.0, 7), (700.0, 0), (6000.0, 31)])
def test_time_domain_weights(A, v, n0):
    """The interpolation weights themselves: a unit impulse gives each output
    one weight.  The curve times are FP64 and the weights are rounded to FP32
    once in the forward (2^-24 of the weight), and at f and again at 1 - f in
    the adjoint (2^-25 each); 1e-11 for the FP64 roundings of T."""
    import torch
    print(f"[gpu] time-domain weights v {v} n0 {n0}", flush=True)
    nt, nx, dt, dx = 300, 40, 0.004, 12.5
    plan = A.Plan(nt, nx, dt, dx, [v], tau0=[n0])
    x, tau = np.arange(nx), np.arange(nt)
    q = (dx / (v * dt)) ** 2
    for xa, ta in [(0, 0), (17, 1), (20, 40), (39, 97), (5, 203), (11, 255)]:
        T = n0 + np.sqrt(ta * ta + (x - xa) ** 2 * q)
        w = np.maximum(0.0, 1.0 - np.abs(T[:, None] - tau[None, :]))
        m = torch.zeros((1, nx, nt), device="cuda")
        m[0, xa, ta] = 1.0
        e = np.abs(plan.td_forward(m).cpu().numpy() - w)
        assert np.all(e <= 2.0 ** -24 * w + 1e-11), e.max()
        i = n0 + ta  # data impulse on trace xa: the times of every apex's curve there
        T = n0 + np.sqrt(tau[None, :] ** 2 + (x - xa)[:, None] ** 2 * q)
        w = np.maximum(0.0, 1.0 - np.abs(T - i))
        d = torch.zeros((nx, nt), device="cuda")
        d[xa, i] = 1.0
        e = np.abs(plan.td_adjoint(d).cpu().numpy()[0] - w)
        assert np.all(e <= 2.0 ** -24 + 1e-11), e.max()
        assert np.all(e[w == 0.0] == 0.0)


# The forward's wider tiles: 8 traces where 32-time by 8-trace tiles number at
# least 512, 4 traces where those of 4 do; ragged times and traces.
@pytest.mark.parametrize("nt,nx,vel,tau0", [(1021, 131, [1500.0], [0]), (509, 131, [1900.0, 0.0], [3, 0]),
                                            (520, 126, [2500.0], [9])])
def test_time_domain_wide_tiles(A, nt, nx, vel, tau0):
    """Same bar as above, with dead traces."""
    import torch
    print(f"[gpu] time-domain wide tiles {nt} x {nx}", flush=True)
    rng = np.random.default_rng(nt)
    m = f32(rng.standard_normal((len(vel), nx, nt)))
    mask = np.ones(nx, np.uint8)
    mask[2::5] = 0
    plan = A.Plan(nt, nx, 0.004, 12.5, vel, tau0=tau0)
    fg = plan.td_forward(torch.tensor(m, dtype=torch.float32, device="cuda"),
                         mask=torch.tensor(mask, device="cuda")).cpu().numpy()
    fr = TD.forward(m[:1], 0.004, 12.5, vel[:1], tau0[:1])
    for p in range(1, len(vel)):
        fr[:, tau0[p]:] += m[p][:, :nt - tau0[p]]  # v = 0
    fr *= mask[:, None]
    assert rel_l2(fg, fr) <= 1e-5


# One tile width each (2, 4 and 8 traces).
@pytest.mark.parametrize("nt,nx", [(90, 21), (509, 131), (1021, 131)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_time_domain_non_finite_sample(A, nt, nx, bad):
    """A model sample that is not finite reaches the outputs on its curve
    (weight above 0) and no other; the adjoint likewise."""
    import torch
    print(f"[gpu] time-domain non-finite sample {nt} x {nx} {bad}", flush=True)
    rng = np.random.default_rng(nx)
    v, xa, ta = 1800.0, nx // 3, nt // 4
    plan = A.Plan(nt, nx, 0.004, 12.5, [v])
    m = torch.tensor(rng.standard_normal((1, nx, nt)), dtype=torch.float32, device="cuda")
    m[0, xa, ta] = 0.0
    f0 = plan.td_forward(m).cpu().numpy()
    m[0, xa, ta] = float(bad)
    f1 = plan.td_forward(m).cpu().numpy()
    T = np.sqrt(ta * ta + (np.arange(nx) - xa) ** 2 * (12.5 / (v * 0.004)) ** 2)
    hit = np.abs(T[:, None] - np.arange(nt)[None, :]) < 1.0
    assert hit.any() and not np.isfinite(f1[hit]).any()
    assert np.array_equal(f1[~hit], f0[~hit])
    d = torch.tensor(rng.standard_normal((nx, nt)), dtype=torch.float32, device="cuda")
    i = nt // 2
    d[xa, i] = 0.0
    a0 = plan.td_adjoint(d).cpu().numpy()[0]
    d[xa, i] = float(bad)
    a1 = plan.td_adjoint(d).cpu().numpy()[0]
    T = np.sqrt(np.arange(nt)[None, :] ** 2 + (np.arange(nx)[:, None] - xa) ** 2 * (12.5 / (v * 0.004)) ** 2)
    # (a curve time on a whole sample reads its later neighbour with weight 0)
    hit = (T >= i - 1) & (T < i + 1)
    assert not np.isfinite(a1[hit]).any()
    assert np.array_equal(a1[~hit], a0[~hit])


# Few waves take 2 apexes and four distances at a time, a full card of them 4
# apexes and two: 75 panels of 130 x 126 (7200 waves of 4) against single ones.
@pytest.mark.parametrize("nt,nx,P", [(130, 126, 75), (129, 127, 75), (64, 250, 114)])
def test_time_domain_adjoint_tiles_agree(A, nt, nx, P):
    """Every tile adds an apex's traces in the same order, so a panel among many
    equals the same panel alone, bit for bit; dead traces hold NaN."""
    import torch
    print(f"[gpu] time-domain adjoint tiles {nt} x {nx} x {P}", flush=True)
    assert (nt + 63) // 64 * ((nx + 3) // 4) * P >= 7168
    rng = np.random.default_rng(nx)
    vel = list(np.linspace(0.0, 5000.0, P))
    tau0 = [int(p % 5 * 3) for p in range(P)]
    mask = (rng.uniform(size=nx) > 0.3).astype(np.uint8)
    for mk in (None, torch.tensor(mask, device="cuda")):
        d = rng.standard_normal((nx, nt))
        if mk is not None:
            d[mask == 0] = np.nan
        d = torch.tensor(d, dtype=torch.float32, device="cuda")
        a = A.Plan(nt, nx, 0.004, 12.5, vel, tau0=tau0).td_adjoint(d, mask=mk).cpu().numpy()
        assert np.isfinite(a).all()
        for p in (0, 1, 17, P // 2, P - 1):
            one = A.Plan(nt, nx, 0.004, 12.5, vel[p:p + 1], tau0=tau0[p:p + 1]).td_adjoint(d, mask=mk).cpu().numpy()
            assert np.array_equal(a[p], one[0]), p

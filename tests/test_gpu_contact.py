"""GPU binning and containment: bit-exact against the FP32 checker on the
GPU's own positions, and equal to the FP64 oracle's decisions except for pairs
whose distance is within 1e-4 rc of the contact radius.

The 1e-4 band: FP32 coordinates near 0.5 mm carry an ulp of 6e-11 m, i.e.
1.2e-5 rc at rc = 5 um; a distance built from three coordinate differences of
positions reconstructed with a few roundings each can move by several ulps."""
import numpy as np
import pytest

from oracle import Oracle, f32_cells, f32_contain
from paper_2504_12858_amd import binding as B
from paper_2504_12858_amd import workloads as W
from tests.gpu_helpers import gpu_parts, ident, orc_parts, require_gpu

pytestmark = pytest.mark.gpu


def _cloud(seed, n_grains, per_grain, lam, m, stopped_frac, spread):
    g = W.rng(seed)
    box = 1e-3
    centre = box / 2 + (g.random((n_grains, 3)) - 0.5) * spread
    quat = W.shoemake_quaternions(g, n_grains)
    grain = np.repeat(np.arange(n_grains, dtype=np.int32), per_grain)
    site = g.integers(-m, m + 1, size=(grain.size, 3)).astype(np.int32)
    d = g.integers(0, 6, size=grain.size).astype(np.int32)
    s = (g.random(grain.size) * lam).astype(np.float32).astype(np.float64)
    state = np.where(g.random(grain.size) < stopped_frac, 1, 0).astype(np.int32)
    # Unique identities (grain, site, dir).
    key = (grain.astype(np.int64) << 40) ^ ((site[:, 0] + 64) << 16) ^ ((site[:, 1] + 64) << 8) ^ (site[:, 2] + 64)
    key = key * 8 + d
    _, first = np.unique(key, return_index=True)
    keep = np.sort(first)
    parts = dict(grain=grain[keep], site=site[keep], dir=d[keep], s=s[keep], state=state[keep])
    return centre, quat, parts


EMPTY_CLAIMS = dict(grain=np.zeros(0, np.int32), site=np.zeros((0, 3), np.int32),
                    flags=np.zeros(0, np.uint8))


@pytest.mark.parametrize("seed,n_grains,per_grain,m,spread,h_factor", [
    (1, 6, 400, 4, 30e-6, 1.0),
    (2, 12, 1500, 8, 60e-6, 1.0),
    (3, 40, 3000, 12, 150e-6, 1.0),   # many 4^3-cell bricks, ragged fill
    (4, 12, 1500, 8, 60e-6, 2.0),     # cells of 2 rc: 2x2x2 stencil
    (5, 40, 3000, 12, 150e-6, 2.0),
])
def test_single_step_contact_parity(seed, n_grains, per_grain, m, spread, h_factor):
    require_gpu()
    lam = 5e-6
    h = h_factor * lam
    dT, dt = 3.0, 1e-4
    centre, quat, parts = _cloud(seed, n_grains, per_grain, lam, m, 0.3, spread)
    print(f"contact parity seed={seed} n={len(parts['grain'])}", flush=True)
    p = B.make_params((0, 0, 0), (1e-3,) * 3, lam, h, lam, W.KIN_A, W.KIN_B, branching=0,
                      cap_particles=1 << 18, cap_stopped=1 << 18, cap_grains=64,
                      cap_claim_bricks=1 << 12)
    ctx = B.Context(p)
    ctx.set_thermal_field(W.Field(W.FIELD_UNIFORM, dT=dT))
    ctx.load_state(centre, quat, parts, EMPTY_CLAIMS, np.zeros(0, np.int32), 0.0, 0)
    ctx.step(dt, 1)
    g, key = gpu_parts(ctx)
    xyz = np.stack([g["x"], g["y"], g["z"]], 1)
    # Binning: exported cells equal single-rounded FP32 binning of the
    # exported positions.
    ncell = int(np.ceil(1e-3 / h))
    cells = f32_cells(xyz, np.zeros(3, np.float32), np.float32(1.0 / h), np.array([ncell] * 3, np.int32))
    np.testing.assert_array_equal(cells, g["cell"])
    # Roles before the step: active particles are tested, stopped ones are obstacles.
    pk = ident(parts["grain"], parts["site"], parts["dir"])
    order = np.argsort(pk)
    np.testing.assert_array_equal(pk[order], key)
    pre_state = parts["state"][order]
    role = np.where(pre_state == 0, 1, 2).astype(np.uint8)
    rc2 = np.float32(lam * lam)
    dec = f32_contain(xyz, g["grain"].astype(np.int32), role, rc2)
    gpu_dec = ((pre_state == 0) & (g["state"] == 1)).astype(np.uint8)
    np.testing.assert_array_equal(gpu_dec, dec)
    assert dec.sum() > 0
    # FP64 oracle: same decisions except pairs within 1e-5 of rc.
    o = Oracle((0, 0, 0), (1e-3,) * 3, lam, h, lam, W.KIN_A, W.KIN_B, branching=0)
    o.set_field(W.Field(W.FIELD_UNIFORM, dT=dT))
    o.load_state(centre, quat, parts, EMPTY_CLAIMS, np.zeros(0, np.int32), 0.0, 0)
    o.step(dt, 1)
    q, okey = orc_parts(o)
    np.testing.assert_array_equal(okey, key)
    assert np.abs(xyz.astype(np.float64) - q["x"]).max() <= 1e-5 * 1e-3
    mism = np.flatnonzero(q["state"] != g["state"])
    for i in mism:
        d = np.sqrt(((q["x"] - q["x"][i]) ** 2).sum(1))
        other = q["grain"] != q["grain"][i]
        near = np.abs(d[other] - lam).min() / lam
        assert near < 1e-4, (i, near)
    assert len(mism) <= 2


@pytest.mark.parametrize("blocks", [1, 8, 100, 2048])
@pytest.mark.parametrize("seed,n_grains,per_grain,m,spread,h_factor", [
    (1, 6, 400, 4, 30e-6, 1.0), (3, 40, 3000, 12, 150e-6, 1.0), (5, 40, 3000, 12, 150e-6, 2.0)])
def test_particles_per_wave_change_no_decision(seed, n_grains, per_grain, m, spread, h_factor, blocks):
    """Crowded clouds (most stencil cells of a particle hold other grains)
    with 8 to 64 particles per wave of the containment, by the blocks of its
    launch, and with more pairs per wave than one round takes: the decisions
    equal the FP32 checker's."""
    require_gpu()
    lam, dt = 5e-6, 1e-4
    centre, quat, parts = _cloud(seed, n_grains, per_grain, lam, m, 0.3, spread)
    p = B.make_params((0, 0, 0), (1e-3,) * 3, lam, h_factor * lam, lam, W.KIN_A, W.KIN_B,
                      branching=0, cap_particles=1 << 18, cap_stopped=1 << 18, cap_grains=64,
                      cap_claim_bricks=1 << 12)
    ctx = B.Context(p)
    ctx.set_schedule({"contain": blocks})
    ctx.set_thermal_field(W.Field(W.FIELD_UNIFORM, dT=3.0))
    ctx.load_state(centre, quat, parts, EMPTY_CLAIMS, np.zeros(0, np.int32), 0.0, 0)
    ctx.step(dt, 1)
    g, key = gpu_parts(ctx)
    order = np.argsort(ident(parts["grain"], parts["site"], parts["dir"]))
    pre_state = parts["state"][order]
    dec = f32_contain(np.stack([g["x"], g["y"], g["z"]], 1), g["grain"].astype(np.int32),
                      np.where(pre_state == 0, 1, 2).astype(np.uint8), np.float32(lam * lam))
    np.testing.assert_array_equal(((pre_state == 0) & (g["state"] == 1)).astype(np.uint8), dec)
    ctx.close()


@pytest.mark.parametrize("blocks", [8, 200, 2048])
def test_full_stopped_store_holds_written_records(blocks):
    """A step that stops twice as many particles as the stopped store has room
    for: the error is reported, and the store is full of particles that were
    stopped before or by this step, each once."""
    require_gpu()
    lam = 5e-6
    centre, quat, parts = _cloud(5, 40, 3000, lam, 12, 0.3, 150e-6)
    loaded = int((parts["state"] == 1).sum())

    def start(cap):
        ctx = B.Context(B.make_params((0, 0, 0), (1e-3,) * 3, lam, 2 * lam, lam, W.KIN_A, W.KIN_B,
                                      branching=0, cap_particles=1 << 18, cap_stopped=cap,
                                      cap_grains=64, cap_claim_bricks=1 << 12))
        ctx.set_schedule({"contain": blocks})
        ctx.set_thermal_field(W.Field(W.FIELD_UNIFORM, dT=3.0))
        ctx.load_state(centre, quat, parts, EMPTY_CLAIMS, np.zeros(0, np.int32), 0.0, 0)
        return ctx
    ctx = start(1 << 18)
    stops = ctx.step(1e-4, 1)["contained"]
    assert stops > 1000
    full, key = gpu_parts(ctx)
    stopped = key[full["state"] == 1]
    ctx.close()
    cap = loaded + stops // 2
    ctx = start(cap)
    with pytest.raises(B.GrainEnvError) as e:
        ctx.step(1e-4, 1)
    assert e.value.status == B.GE_ECAPACITY
    q = ctx.particles()
    q = q[q["state"] == 1]
    got = ident(q["grain"], q["site"], q["dir"])
    assert len(got) == cap == len(np.unique(got))
    assert np.isin(got, stopped).all()
    # The context is usable again with a state that fits.
    ctx.load_state(centre, quat, {k: v[:100] for k, v in parts.items()}, EMPTY_CLAIMS,
                   np.zeros(0, np.int32), 0.0, 0)
    assert ctx.step(1e-4, 1)["step"] == 1
    ctx.close()


def test_stopped_particles_block_and_survive_steps():
    """A stopped wall of grain 0 stops grain 1's particles arriving later."""
    require_gpu()
    lam = 5e-6
    p = B.make_params((0, 0, 0), (1e-3,) * 3, lam, lam, lam, W.KIN_A, W.KIN_B, branching=0,
                      cap_particles=1024, cap_stopped=1024, cap_grains=4, cap_claim_bricks=1024)
    ctx = B.Context(p)
    ctx.set_thermal_field(W.Field(W.FIELD_UNIFORM, dT=5.0))
    gap0 = 20.3e-6   # (gap0 - rc) / (v dt) is not an integer: no tie at the meeting step
    c = np.array([[5e-4, 5e-4, 5e-4], [5e-4 - gap0, 5e-4, 5e-4]])
    q = np.array([[1.0, 0, 0, 0]] * 2)
    parts = dict(grain=np.array([0, 1], np.int32), site=np.zeros((2, 3), np.int32),
                 dir=np.array([1, 0], np.int32), s=np.zeros(2), state=np.array([1, 0], np.int32))
    ctx.load_state(c, q, parts, EMPTY_CLAIMS, np.zeros(0, np.int32), 0.0, 0)
    v = 1e-5 * 25 + 1e-6 * 125
    n_meet = int(np.floor((gap0 - lam) / (v * 1e-4))) + 1
    ctx.step(1e-4, n_meet - 1)
    assert ctx.counts()["n_active"] == 1
    ctx.step(1e-4, 1)
    st = ctx.counts()
    assert st["n_active"] == 0 and st["n_stopped"] == 2


@pytest.mark.parametrize("seed,n_grains,per_grain,m,spread,h_factor,periodic", [
    (6, 12, 60, 6, 120e-6, 1.0, 0), (7, 12, 60, 6, 120e-6, 2.0, 0),   # several bricks per stencil
    (8, 40, 400, 8, 150e-6, 2.0, 0),                                  # crowded bricks
    (9, 12, 60, 6, 120e-6, 1.0, 7), (10, 12, 60, 6, 120e-6, 2.0, 7)])  # around a periodic corner
def test_sites_near_particles_do_not_fire(seed, n_grains, per_grain, m, spread, h_factor, periodic):
    """Sites of a cloud without claims: one fires unless a particle or an
    earlier site fired in the step lies within rc, in the FP32 arithmetic of
    the step on its own exported positions."""
    require_gpu()
    lam = 5e-6
    f4 = np.float32
    centre, quat, parts = _cloud(seed, n_grains, per_grain, lam, m, 0.3, spread)
    g = W.rng(seed + 100)
    sites = 5e-4 + (g.random((600, 3)) - 0.5) * (spread + 2 * m * lam)
    if periodic:
        centre, sites = centre - 5e-4, np.mod(sites - 5e-4, 1e-3)
    p = B.make_params((0, 0, 0), (1e-3,) * 3, lam, h_factor * lam, lam, W.KIN_A, W.KIN_B,
                      branching=0, cap_particles=1 << 16, cap_stopped=1 << 16, cap_grains=1024,
                      cap_claim_bricks=1 << 12, cap_sites=1024, periodic=periodic)
    ctx = B.Context(p)
    ctx.set_thermal_field(W.Field(W.FIELD_UNIFORM, dT=3.0))
    ctx.load_state(centre, quat, parts, EMPTY_CLAIMS, np.zeros(0, np.int32), 0.0, 0)
    ctx.nucleate(sites, np.zeros(len(sites)), W.shoemake_quaternions(g, len(sites)))
    ctx.step(1e-4, 1)
    q = ctx.particles()
    q = q[q["grain"] < n_grains]
    x = np.stack([q["x"], q["y"], q["z"]], 1).astype(f4)
    y = sites.astype(f4)
    L = f4(1e-3)

    def near(a, b):
        d = a - b
        if periodic:  # nearest images; the product is exact in FP64, so one rounding
            k = np.rint(d * (f4(1) / L))
            d = (d.astype(np.float64) - k.astype(np.float64) * np.float64(L)).astype(f4)
        return (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2] < f4(lam * lam)

    want = np.zeros(len(y), bool)
    for i in range(len(y)):
        want[i] = not near(y[i], x).any() and not (want.any() and near(y[i], y[want]).any())
    assert 20 < want.sum() < len(y) - 20
    np.testing.assert_array_equal(ctx.site_states() == 1, want)
    ctx.close()

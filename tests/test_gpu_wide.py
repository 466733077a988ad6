"""GPU parity of the large-Nc path (one workgroup per link, link-major
storage) against the FP64 oracle, for 4 <= Nc <= 32.

The tolerances are those of test_gpu_parity (K_LINK eps (1 + c) per link,
FP32 decision flips inside K_FLIP eps (1 + c) counted), widened where the
oracle itself is sensitive: one link update is a chain of Nc (Nc - 1) / 2
subgroup steps (496 at Nc = 32), each dividing by its own k, so rounding
compounds along the chain.  The oracle's phase is run three more times with
its input perturbed at the storage precision's rounding level (1e-7 FP32,
1e-15 FP64), and a link may differ by up to SPREAD_FACTOR times the largest
change those perturbations make to it (10 in FP64, 100 in FP32: the FP32
arithmetic along the chain adds rounding at every step, which an input
perturbation does not model)."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_common import (EPS, K_FLIP, K_TYP, TOL, beta_for, compare_links, gpu_lattice, oracle_phase_diag,
                        record, rounded, thermal_field, to_np, twin_spread)

pytestmark = pytest.mark.gpu

SMALL = (4, 4, 2, 2)      # V/2 = 32 links per phase
REL = {"f32": 1e-7, "f64": 1e-15}   # input perturbation of the oracle twin


@pytest.mark.parametrize("nc,dtype", [(4, "f64w"), (4, "f32w"), (5, "f32"), (9, "f64"), (9, "f32"), (16, "f64"),
                                      (16, "f32"), (28, "f64"), (32, "f64"), (32, "f32")])
def test_wide_hot_start_parity(gpu, nc, dtype):
    L = (4, 2, 2, 2)
    lat = gpu_lattice(gpu, nc, L, dtype, hot=True, seed=1234)
    got = to_np(lat.export())
    want = O.new_field(nc, L, hot=True, seed=1234)
    # Gram-Schmidt of an Nc x Nc Gaussian matrix: rounding ~ cond(M) eps
    tol = 1e-11 if dtype.startswith("f64") else 1e-6
    assert np.abs(got - want).max() < tol


@pytest.mark.parametrize("nc", [4, 10])
def test_wide_cold_start_exact(gpu, nc):
    lat = gpu_lattice(gpu, nc, (4, 4, 2, 2), "f32w", hot=False)
    assert np.array_equal(to_np(lat.plaquette()), [1.0, 1.0, 1.0])
    assert np.array_equal(to_np(lat.polyakov()), [1.0, 0.0])
    assert np.array_equal(to_np(lat.unitarity()), [0.0, 0.0])


@pytest.mark.parametrize("nc,dtype", [(5, "f64w"), (12, "f32"), (12, "f64")])
def test_wide_roundtrip(gpu, nc, dtype):
    L = (4, 2, 2, 2)
    U = O.new_field(nc, L, hot=True, seed=5)
    lat = gpu_lattice(gpu, nc, L, dtype, field=U)
    assert np.array_equal(to_np(lat.export()), rounded(U, dtype))


@pytest.mark.parametrize("nc,dtype", [(4, "f64w"), (9, "f64"), (9, "f32"), (13, "f64"), (16, "f64"), (32, "f32")])
def test_wide_observables_parity(gpu, nc, dtype):
    L = (4, 2, 2, 4)
    lat = gpu_lattice(gpu, nc, L, dtype, field=thermal_field(nc, L, beta_for(nc), sweeps=1))
    U = to_np(lat.export())
    np.testing.assert_allclose(to_np(lat.plaquette()), O.plaquette(U, nc, L), rtol=1e-13, atol=1e-15)
    pg = to_np(lat.polyakov())
    assert abs(complex(pg[0], pg[1]) - O.polyakov(U, nc, L)) < 1e-13
    np.testing.assert_allclose(to_np(lat.unitarity()), O.unitarity(U, nc, L), rtol=1e-6, atol=1e-14)


@pytest.mark.parametrize("nc,noise,tol", [(4, 1e-3, 1e-12), (9, 1e-3, 1e-12), (16, 1e-3, 1e-12), (32, 1e-3, 1e-12),
                                          (9, 1.0, 1e-10), (16, 1.0, 1e-10), (32, 1.0, 1e-10)])
def test_wide_reunitarize_parity(gpu, nc, noise, tol):
    """Near-unitary links (noise 1e-3: one Gram-Schmidt pass per row) and
    general ones (noise 1: the later rows lose more than half their norm to
    the projection and take the second pass); the latter agree with the
    oracle to the conditioning of a random matrix times the unit roundoff."""
    L = (4, 2, 2, 2)
    rng = np.random.default_rng(nc)
    U = O.new_field(nc, L, hot=True, seed=9)
    U = U + noise * (rng.standard_normal(U.shape) + 1j * rng.standard_normal(U.shape))
    lat = gpu_lattice(gpu, nc, L, "f64" if nc > 8 else "f64w", field=U)
    before = to_np(lat.reunitarize(report=True))
    after = to_np(lat.export())
    np.testing.assert_allclose(before, O.unitarity(U, nc, L), rtol=1e-10)
    O.reunitarize(U, nc, L)
    assert np.abs(after - U).max() < tol
    assert to_np(lat.unitarity()).max() < 1e-13


PHASES = [(0, 0, 0), (0, 3, 1), (1, 1, 1), (1, 2, 0)]   # (kind, mu, parity)


@pytest.mark.parametrize("nc,dtype", [(4, "f64w"), (4, "f32w"), (5, "f64w"), (9, "f64"), (9, "f32"),
                                      (16, "f64"), (16, "f32"), (24, "f64"), (32, "f64"), (32, "f32"),
                                      (21, "f32"), (27, "f32"),    # matrix-core products on ragged tiles
                                      (30, "f32")])                # with the staple sum in registers
def test_wide_phase_parity(gpu, nc, dtype):
    beta = beta_for(nc)
    base = thermal_field(nc, SMALL, beta, sweeps=1) if nc <= 16 else O.new_field(nc, SMALL, hot=True, seed=21)
    lat = gpu_lattice(gpu, nc, SMALL, dtype, field=base)
    flips = 0
    for kind, mu, par in PHASES:
        before = to_np(lat.export())               # the GPU's own input field
        lat.phase(kind, mu, par, beta, seed=77, step=3)
        got = to_np(lat.export())
        sp = twin_spread(before, nc, SMALL, kind, mu, par, beta, 77, 3, rel=REL[dtype[:3]])
        want = before.copy()
        m, k = oracle_phase_diag(want, nc, SMALL, kind, mu, par, beta, 77, 3)
        dec = (np.prod(SMALL) // 2) * nc * (nc - 1) // 2 if kind == 0 else None
        flips += compare_links(got, want, dtype, m, k, f"nc={nc} {dtype} kind={kind} mu={mu} p={par}", spread=sp,
                               decisions=dec)
    print(f"flips: {flips}")


def test_wide_su32_8x4_phase_parity(gpu):
    """The paper's largest single-precision case: SU(32) on 8^4."""
    nc, L, beta = 32, (8, 8, 8, 8), 6.2
    lat = gpu_lattice(gpu, nc, L, "f32", hot=True, seed=1234)
    base = to_np(lat.export())
    lat.phase(0, 1, 0, beta, seed=1234, step=0)
    got = to_np(lat.export())
    sp = twin_spread(base, nc, L, 0, 1, 0, beta, 1234, 0, rel=REL["f32"])
    m, k = oracle_phase_diag(base, nc, L, 0, 1, 0, beta, 1234, 0)
    flips = compare_links(got, base, "f32", m, k, "SU(32) 8^4 heatbath", spread=sp,
                          decisions=(8 ** 4 // 2) * nc * (nc - 1) // 2)
    print(f"flips: {flips}")


@pytest.mark.parametrize("dtype", ["f64w", "f32w"])
def test_wide_batched_sampler_parity(gpu, dtype):
    """The large-Nc draw, batched over eight subgroups with the fall-back to
    attempts 8..63, against the oracle's sequential sampler on the same
    counters (element i: subgroup mu_sg + i mod 8 of site i / 8).  Near
    alpha = 1.7, the hybrid's lowest acceptance, some draws need more than
    eight attempts on either side of the switch and so take the fall-back."""
    sun = gpu
    alpha = np.concatenate([np.zeros(64), np.linspace(0.01, 60.0, 40000), np.full(160000, 1.7),
                            np.full(160000, 1.69)])
    mu_sg = (2 << 16) | 8
    xg, ag = sun.sample_su2(torch.from_numpy(alpha).cuda(), seed=31, step=5, mu_sg=mu_sg, dtype=dtype)
    xg, ag = to_np(xg), to_np(ag)
    xo, ao, margin = np.zeros((alpha.size, 4)), np.zeros(alpha.size, dtype=np.int32), np.zeros(alpha.size)
    for s in range(8):
        xo[s::8], ao[s::8], margin[s::8] = O.sample_su2(alpha[s::8], seed=31, step=5, mu_sg=mu_sg + s)
    assert (ao[alpha == 1.7] > 8).sum() > 0 and (ao[alpha == 1.69] > 8).sum() > 0
    d = np.abs(xg - xo).max(axis=1)
    bad = (d > TOL[dtype]) | (ag != ao)
    ok = ~bad
    record(what="batched sampler", dtype=dtype, links=int(d.size), max_dU=float(d[ok].max()),
           max_dU_over_tol=float(d[ok].max() / TOL[dtype]), flips=int(bad.sum()),
           flip_margins=[float(m) for m in margin[bad][:50]])
    if dtype == "f64w":
        assert not bad.any(), (d.max(), int((ag != ao).sum()))
    else:
        # as check_draw_flips of the register-path sampler test
        eps = EPS["f32"]
        assert np.all(margin[bad] < K_FLIP * eps * (1.0 + alpha[bad]))
        expected = float((2 * 2 * K_TYP * eps * (1.0 + alpha)).sum())
        assert bad.sum() <= max(3.0, 3.0 * expected), (int(bad.sum()), expected)


@pytest.mark.parametrize("nc", [4])
def test_wide_agrees_with_register_path(gpu, nc):
    """The two implementations of SU(4) draw the same random numbers: a
    heatbath and an overrelaxation phase agree to FP64 rounding."""
    L = (4, 4, 2, 2)
    U = thermal_field(nc, L, beta_for(nc), sweeps=1)
    a = gpu_lattice(gpu, nc, L, "f64", field=U)
    b = gpu_lattice(gpu, nc, L, "f64w", field=U)
    for lat in (a, b):
        lat.phase(0, 2, 1, beta_for(nc), seed=5, step=1)
        lat.phase(1, 0, 0, beta_for(nc), seed=5, step=1)
    assert np.abs(to_np(a.export()) - to_np(b.export())).max() < 1e-11
    np.testing.assert_allclose(to_np(a.plaquette()), to_np(b.plaquette()), rtol=1e-13)


def test_wide_sweep_is_its_phase_sequence(gpu):
    nc, L = 10, (4, 4, 2, 2)
    beta = beta_for(nc)
    a = gpu_lattice(gpu, nc, L, "f32", hot=True, seed=4)
    b = gpu_lattice(gpu, nc, L, "f32", hot=True, seed=4)
    a.sweep(beta, 1, 2, seed=4)
    for kind, steps in ((0, 1), (1, 2)):
        for _ in range(steps):
            for mu in range(4):
                for par in range(2):
                    b.phase(kind, mu, par, beta, seed=4, step=0)
    b.reunitarize()
    assert torch.equal(a.links, b.links)
    assert a.step == 1


@pytest.mark.parametrize("nc,dtype", [(9, "f32"), (16, "f32"), (20, "f32"), (12, "f64"), (26, "f64"), (32, "f64"),
                                      (24, "f32")])
def test_wide_one_or_two_wavefronts_give_the_same_bits(gpu, nc, dtype):
    """A link's update on one wavefront (launch block 64), on two (block
    128: loads and vector-unit products shared by row groups) and with the
    default choice give the same field bit for bit, heatbath and
    overrelaxation (at Nc = 24 in FP32 the matrix-core products stay on the
    first wavefront and the second shares the loads)."""
    sun = gpu
    L, beta = (4, 4, 2, 2), beta_for(nc)
    base = O.new_field(nc, L, hot=True, seed=41)
    fields = []
    for block in (64, 128, 256):
        lat = gpu_lattice(sun, nc, L, dtype, field=base)
        lat.set_launch(block)
        for kind, mu, par in [(0, 1, 0), (1, 2, 1), (0, 3, 1), (1, 0, 0)]:
            lat.phase(kind, mu, par, beta, seed=5, step=3)
        torch.cuda.synchronize()
        fields.append(lat.links.clone())
    assert torch.equal(fields[0], fields[1])
    assert torch.equal(fields[0], fields[2])


def test_wide_field_past_4_gib_phase_parity(gpu):
    """The workgroup-per-link path on a field larger than 4 GiB (SU(8) FP64
    on 32^3 x 34: 4.6 GB), so that link addresses pass 2^32 bytes: a heatbath
    phase of direction 3 (the top of the field) link by link against the
    oracle, the other directions unchanged bit for bit."""
    nc, L, dtype, seed = 8, (32, 32, 32, 34), "f64", 99
    beta = beta_for(nc)
    lat = gpu_lattice(gpu, nc, L, dtype, hot=True, seed=seed)
    assert lat.links.numel() * lat.links.element_size() > 2 ** 32
    before = to_np(lat.export())
    lat.phase(0, 3, 1, beta, seed=seed, step=0)
    got = to_np(lat.export())
    for mu in range(3):
        assert np.array_equal(got[mu], before[mu]), mu
    sp = twin_spread(before, nc, L, 0, 3, 1, beta, seed, 0, rel=REL["f64"], twins=1)
    m, k = oracle_phase_diag(before, nc, L, 0, 3, 1, beta, seed, 0)
    compare_links(got[3:], before[3:], dtype, m[3:], k[3:], "SU(8) 32^3x34 kind 0 mu 3 p 1", spread=sp[3:])


WIDE_BATCH = [  # (nc, L, dtype, beta, seed)
    (5, (4, 4, 2, 2), "f32", beta_for(5), 21),
    (5, (4, 2, 4, 2), "f32", beta_for(5) + 0.7, 22),    # same group, other extents and coupling
    (8, (4, 4, 2, 2), "f64", beta_for(8), 23),
    (4, (4, 4, 2, 2), "f32w", 11.1, 24),                # SU(4) on the workgroup-per-link path
    (3, (4, 4, 4, 4), "f32", 6.0, 25),                  # a register-path chain in the same batch
    (6, (4, 4, 1, 4), "f64", beta_for(6), 26),          # 3D: an absent direction
    (24, (4, 2, 2, 2), "f32", beta_for(24), 27),        # matrix-core products
    (22, (2, 2, 4, 2), "f64", beta_for(22), 28),        # staple sum in registers
    (12, (4, 2, 2, 4), "f32", beta_for(12), 29),        # two wavefronts per link
    (26, (2, 2, 2, 4), "f64", beta_for(26), 30),        # two wavefronts for the overrelaxation
]


def test_wide_chains_in_a_batch_are_bitwise_the_chains_alone(gpu):
    """Large-Nc chains join a batch (one launch per phase for each Nc and
    precision): two eager sweeps, then a captured sweep replayed three times
    with eager work between the replays, give bitwise the fields and
    plaquettes of the chains swept alone, and the step counters advance
    alike."""
    sun = gpu
    alone = [gpu_lattice(sun, nc, L, dt, hot=True, seed=sd) for nc, L, dt, b, sd in WIDE_BATCH]
    batched = [gpu_lattice(sun, nc, L, dt, hot=True, seed=sd) for nc, L, dt, b, sd in WIDE_BATCH]
    for lat, (nc, L, dt, beta, sd) in zip(alone, WIDE_BATCH):
        for _ in range(5):
            lat.sweep(beta, 1, 2, seed=sd)
    bt = sun.Batch(batched, [c[3] for c in WIDE_BATCH], [c[4] for c in WIDE_BATCH])
    bt.sweep(1, 2)
    bt.sweep(1, 2)
    plaq = torch.zeros((len(WIDE_BATCH), 3), dtype=torch.float64, device="cuda")
    bt.capture(n_sweeps=1, n_hb=1, n_or=2, plaq_out=plaq)
    for _ in range(3):
        bt.replay()
        torch.cuda.synchronize()
        _ = bt.plaquette()
        torch.cuda.synchronize()
    bt.sync()
    for i, (a, b) in enumerate(zip(alone, batched)):
        assert torch.equal(a.links, b.links), f"chain {i} {WIDE_BATCH[i][:3]} differs"
        assert a.step == b.step == 5
        assert torch.equal(a.plaquette(), plaq[i]), f"plaquette of chain {i}"
        assert torch.equal(a.plaquette(), bt.plaquette()[i]), f"eager batch plaquette of chain {i}"
    # the batch's launch block reaches its large-Nc groups too (64: one
    # wavefront per link, 128: two), with the same bits
    for block in (64, 128):
        again = [gpu_lattice(sun, nc, L, dt, hot=True, seed=sd) for nc, L, dt, b, sd in WIDE_BATCH]
        bb = sun.Batch(again, [c[3] for c in WIDE_BATCH], [c[4] for c in WIDE_BATCH])
        bb.set_launch(block)
        for _ in range(5):
            bb.sweep(1, 2)
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(alone, again)):
            assert torch.equal(a.links, b.links), f"block {block}: chain {i} {WIDE_BATCH[i][:3]} differs"


def test_wide_batch_couplings_from_a_device_array(gpu):
    """As the register path's coupling-array test, for a batch of large-Nc
    chains: a graph replay reads the coupling array's contents at that
    time."""
    sun = gpu
    cfg = WIDE_BATCH[:4]
    b1 = torch.tensor([c[3] + 0.3 for c in cfg], dtype=torch.float64, device="cuda")
    b2 = torch.tensor([c[3] - 0.2 for c in cfg], dtype=torch.float64, device="cuda")
    alone = [gpu_lattice(sun, nc, L, dt, hot=True, seed=sd) for nc, L, dt, b, sd in cfg]
    batched = [gpu_lattice(sun, nc, L, dt, hot=True, seed=sd) for nc, L, dt, b, sd in cfg]
    for i, (lat, (nc, L, dt, beta, sd)) in enumerate(zip(alone, cfg)):
        for bb in (b1, b2, b1):
            lat.sweep(float(bb[i]), 1, 1, seed=sd)
    bt = sun.Batch(batched, [c[3] for c in cfg], [c[4] for c in cfg])
    bt.sweep(1, 1, beta=b1)
    arr = b2.clone()
    bt.capture(n_sweeps=1, n_hb=1, n_or=1, beta=arr)
    bt.replay()
    torch.cuda.synchronize()
    arr.copy_(b1)
    torch.cuda.synchronize()
    bt.replay()
    torch.cuda.synchronize()
    bt.sync()
    for i, (a, b) in enumerate(zip(alone, batched)):
        assert torch.equal(a.links, b.links), f"chain {i} differs"


@pytest.mark.parametrize("nc,dtype,L", [(5, "f64", (4, 4, 1, 4)), (9, "f32", (4, 2, 4, 1)), (6, "f64", (4, 1, 4, 1))])
def test_wide_absent_direction(gpu, nc, dtype, L):
    """3D and 2D lattices: links of an absent direction stay the identity,
    the staple has 2(d-1) terms, and the observables normalise over the
    planes that exist."""
    beta = beta_for(nc)
    base = O.new_field(nc, L, hot=True, seed=31)
    lat = gpu_lattice(gpu, nc, L, dtype, field=base)
    for kind, mu, par in [(0, 0, 1), (1, 1, 0), (0, 3 if L[3] > 1 else 2, 0)]:
        before = to_np(lat.export())
        lat.phase(kind, mu, par, beta, seed=3, step=2)
        got = to_np(lat.export())
        sp = twin_spread(before, nc, L, kind, mu, par, beta, 3, 2, rel=REL[dtype[:3]])
        want = before.copy()
        m, k = oracle_phase_diag(want, nc, L, kind, mu, par, beta, 3, 2)
        compare_links(got, want, dtype, m, k, f"3D nc={nc} kind={kind} mu={mu}", spread=sp)
    U = to_np(lat.export())
    absent = [d for d in range(4) if L[d] == 1][0]
    assert np.array_equal(U[absent], np.broadcast_to(np.eye(nc), U[absent].shape))
    np.testing.assert_allclose(to_np(lat.plaquette()), O.plaquette(U, nc, L), rtol=1e-13, atol=1e-15)
    pg = to_np(lat.polyakov())
    assert abs(complex(pg[0], pg[1]) - O.polyakov(U, nc, L)) < 1e-13


@pytest.mark.parametrize("nc,dtype", [(4, "f64"), (4, "f64w"), (6, "f64"), (12, "f64"), (32, "f64")])
def test_wide_permutation_links_need_pivoting(gpu, nc, dtype):
    """Links that are permutation matrices times phases: every column of the
    LU elimination has a single nonzero below the pivot row, so the
    determinant depends on the row exchanges (and on the first largest pivot
    among zeros).  Re-unitarization and the unitarity report must match the
    oracle (SU(4) also on the register path, whose determinant pivots the
    same way)."""
    L = (4, 2, 2, 2)
    rng = np.random.default_rng(nc)
    V = int(np.prod(L))
    U = np.zeros((4, V, nc, nc), dtype=np.complex128)
    for mu in range(4):
        for s in range(V):
            perm = rng.permutation(nc)
            U[mu, s, np.arange(nc), perm] = np.exp(1j * rng.uniform(-np.pi, np.pi, nc))
    lat = gpu_lattice(gpu, nc, L, dtype, field=U)
    np.testing.assert_allclose(to_np(lat.unitarity()), O.unitarity(U, nc, L), rtol=1e-10, atol=1e-14)
    lat.reunitarize()
    O.reunitarize(U, nc, L)
    assert np.abs(to_np(lat.export()) - U).max() < 1e-13
    assert to_np(lat.unitarity()).max() < 1e-13


@pytest.mark.parametrize("L", [(6, 2, 1, 1), (2, 2, 2, 2), (6, 2, 4, 2)])   # 6, 8 and 48 links per phase
@pytest.mark.parametrize("nc,dtype", [(4, "f32w"), (4, "f64w"), (5, "f32"), (5, "f64"), (6, "f32"), (6, "f64"),
                                      (7, "f32"), (7, "f64"), (8, "f32"), (8, "f64")])
def test_wide_four_links_per_wavefront(gpu, nc, dtype, L):
    """Up to Nc = 8 a wavefront updates four links: every Nc of that form,
    with a last wavefront that is not full, and with a coupling so small that
    the draws take the Creutz range and attempts past a record's four."""
    base = O.new_field(nc, L, hot=True, seed=51)
    lat = gpu_lattice(gpu, nc, L, dtype, field=base)
    for kind, mu, par, beta in [(0, 0, 1, beta_for(nc)), (0, 1, 0, 0.3 * nc), (1, 1, 1, 1.0), (1, 0, 0, 1.0)]:
        before = to_np(lat.export())
        lat.phase(kind, mu, par, beta, seed=13, step=4)
        got = to_np(lat.export())
        sp = twin_spread(before, nc, L, kind, mu, par, beta, 13, 4, rel=REL[dtype[:3]])
        want = before.copy()
        m, k = oracle_phase_diag(want, nc, L, kind, mu, par, beta, 13, 4)
        compare_links(got, want, dtype, m, k, f"nc={nc} {dtype} kind={kind} beta={beta}", spread=sp)


@pytest.mark.parametrize("nc,dtype", [(10, "f32"), (15, "f64"), (17, "f32"), (17, "f64"), (20, "f32"), (25, "f32"),
                                      (25, "f64"), (26, "f32"), (26, "f64"), (31, "f32"), (31, "f64")])
def test_wide_two_wavefronts_at_the_edges_of_their_ranges(gpu, nc, dtype):
    """From Nc = 9 a link has two wavefronts and matrix-core tiles: the first
    and last Nc of each tile form, odd ones (whose products end on a padded
    k) among them, and a coupling in the draws' Creutz range."""
    L = (4, 2, 2, 2)
    base = O.new_field(nc, L, hot=True, seed=61)
    lat = gpu_lattice(gpu, nc, L, dtype, field=base)
    for kind, mu, par, beta in [(0, 0, 1, beta_for(nc)), (0, 1, 0, 0.3 * nc), (1, 3, 1, 1.0)]:
        before = to_np(lat.export())
        lat.phase(kind, mu, par, beta, seed=17, step=6)
        got = to_np(lat.export())
        sp = twin_spread(before, nc, L, kind, mu, par, beta, 17, 6, rel=REL[dtype[:3]])
        want = before.copy()
        m, k = oracle_phase_diag(want, nc, L, kind, mu, par, beta, 17, 6)
        dec = (np.prod(L) // 2) * nc * (nc - 1) // 2 if kind == 0 else None
        compare_links(got, want, dtype, m, k, f"nc={nc} {dtype} kind={kind} beta={beta}", spread=sp, decisions=dec)


@pytest.mark.parametrize("nc,dtype", [(19, "f32"), (19, "f64"), (20, "f64")])
def test_wide_three_entries_to_a_lane(gpu, nc, dtype):
    """The last Nc of the form with three entries of a link to a lane, and the
    first past it."""
    test_wide_two_wavefronts_at_the_edges_of_their_ranges(gpu, nc, dtype)


@pytest.mark.parametrize("nc,dtype", [(6, "f32"), (8, "f64"), (9, "f32"), (22, "f64"), (23, "f64")])
@pytest.mark.parametrize("scale", [0.02, 0.3])
def test_wide_heatbath_in_the_creutz_range(gpu, nc, dtype, scale):
    """Couplings at which most draws are in the Creutz range and many reject
    their attempts on record (two or three of them), on either side of the
    Nc from which the FP64 heatbath takes the largest form."""
    L = (4, 2, 2, 2)
    base = O.new_field(nc, L, hot=True, seed=67)
    lat = gpu_lattice(gpu, nc, L, dtype, field=base)
    lat.phase(0, 2, 1, scale * nc, seed=19, step=3)
    got = to_np(lat.export())
    sp = twin_spread(base, nc, L, 0, 2, 1, scale * nc, 19, 3, rel=REL[dtype[:3]])
    want = base.copy()
    m, k = oracle_phase_diag(want, nc, L, 0, 2, 1, scale * nc, 19, 3)
    compare_links(got, want, dtype, m, k, f"nc={nc} {dtype} creutz", spread=sp,
                  decisions=(np.prod(L) // 2) * nc * (nc - 1) // 2)


@pytest.mark.parametrize("nc", [25, 26, 32])
@pytest.mark.parametrize("scale", [0.02, 0.3])
def test_wide_heatbath_with_three_creutz_words(gpu, nc, scale):
    """Records whose three attempts serve the Creutz range (FP64, the largest
    form), on both sides of its odd and even Nc."""
    test_wide_heatbath_in_the_creutz_range(gpu, nc, "f64", scale)


@pytest.mark.parametrize("nc,dtype,L", [(5, "f32", (6, 2, 1, 2)), (6, "f64", (2, 2, 2, 2)), (7, "f32", (4, 2, 2, 2)),
                                        (8, "f64", (6, 2, 1, 1)), (12, "f32", (4, 2, 2, 2)), (17, "f64", (2, 2, 2, 2)),
                                        (20, "f32", (2, 2, 2, 2)), (25, "f64", (2, 2, 1, 2)), (31, "f32", (2, 2, 2, 2))])
def test_wide_plaquette_of_every_tile_form(gpu, nc, dtype, L):
    """The plaquette where four sites share a wavefront (Nc <= 8), on one
    tile (<= 16) and on four, odd Nc and absent directions among them."""
    lat = gpu_lattice(gpu, nc, L, dtype, field=thermal_field(nc, L, beta_for(nc), sweeps=1))
    U = to_np(lat.export())
    np.testing.assert_allclose(to_np(lat.plaquette()), O.plaquette(U, nc, L), rtol=1e-13, atol=1e-15)


@pytest.mark.parametrize("nc,noise", [(5, 1e-3), (6, 1e-3), (7, 1e-3), (8, 1e-3), (12, 1e-3), (13, 1e-3), (17, 1e-3),
                                      (24, 1e-3), (25, 1e-3), (6, 1.0), (8, 1.0), (13, 1.0), (25, 1.0)])
def test_wide_reunitarize_row_layouts(gpu, nc, noise):
    """Re-unitarization at the first and last Nc of each row layout (8, 16 or
    32 lanes a row), near-unitary links and general ones (second pass), with
    the deviations found before; and the same bits without the report.  The
    tolerances are those of test_wide_reunitarize_parity."""
    L = (2, 2, 2, 2)
    rng = np.random.default_rng(100 + nc)
    U = O.new_field(nc, L, hot=True, seed=19)
    U = U + noise * (rng.standard_normal(U.shape) + 1j * rng.standard_normal(U.shape))
    lat, plain = (gpu_lattice(gpu, nc, L, "f64w", field=U) for _ in range(2))
    before = to_np(lat.reunitarize(report=True))
    plain.reunitarize()
    after = to_np(lat.export())
    assert torch.equal(lat.links, plain.links)
    np.testing.assert_allclose(before, O.unitarity(U, nc, L), rtol=1e-10)
    O.reunitarize(U, nc, L)
    assert np.abs(after - U).max() < (1e-12 if noise < 1 else 1e-10)
    assert to_np(lat.unitarity()).max() < 1e-13


@pytest.mark.parametrize("nc,dtype,L", [(17, "f32", (4, 4, 8, 8)), (17, "f64", (4, 4, 8, 8)), (18, "f64", (32, 32, 1, 1)),
                                        (18, "f32", (16, 8, 1, 8)), (19, "f32", (4, 4, 8, 8)), (20, "f64", (10, 16, 4, 4)),
                                        (20, "f32", (10, 16, 4, 4)), (19, "f64", (4, 4, 4, 14)), (20, "f32", (4, 2, 2, 2)),
                                        (21, "f32", (2, 2, 2, 2))])
def test_wide_plaquette_rows_and_columns_past_a_tile(gpu, nc, dtype, L):
    """Nc = 17 ... 20 from four (Nc = 20: ten) sites per CU on: one tile and its
    rows and columns past 15 (33, 68, 105 and 144 entries); just below that and
    at Nc = 21 the four tiles."""
    lat = gpu_lattice(gpu, nc, L, dtype, hot=True, seed=71)
    U = to_np(lat.export())
    np.testing.assert_allclose(to_np(lat.plaquette()), O.plaquette(U, nc, L), rtol=1e-13, atol=1e-15)
    # the same bits in a batch beside small and large chains
    others = [gpu_lattice(gpu, nc, E, dtype, hot=True, seed=72) for E in ((2, 2, 2, 2), (8, 8, 8, 6))]
    bt = gpu.Batch([others[0], lat, others[1]], [1.0] * 3, [1, 2, 3])
    for got, chain in zip(to_np(bt.plaquette()), (others[0], lat, others[1])):
        assert np.array_equal(got, to_np(chain.plaquette()))


@pytest.mark.parametrize("nc,noise", [(18, 1e-3), (19, 1e-3), (17, 1.0), (18, 1.0)])
def test_wide_reunitarize_nine_columns(gpu, nc, noise):
    """The layout with nine columns to a lane, to its last Nc and past it."""
    test_wide_reunitarize_row_layouts(gpu, nc, noise)


@pytest.mark.parametrize("nc,dtype", [(4, "f64w"), (5, "f32"), (6, "f64"), (8, "f32"), (12, "f64"), (13, "f32"),
                                      (16, "f64"), (25, "f32"), (32, "f64")])
def test_wide_singular_links_have_determinant_zero(gpu, nc, dtype):
    """A link that is exactly singular -- all zero, or with a zero first, middle
    or last column -- has det U = 0, so both deviations are exactly 1 as the
    oracle's are, wherever the link stands among those of its wavefront; and
    re-unitarization gives every other link the bits it has without it."""
    L = (2, 2, 2, 2)
    base = O.new_field(nc, L, hot=True, seed=23)
    good = gpu_lattice(gpu, nc, L, dtype, field=base)
    good.reunitarize()
    want = to_np(good.export())
    cols = {"zero": slice(None), "first": 0, "middle": nc // 2, "last": nc - 1}
    for k, (what, col) in enumerate(cols.items()):
        mu, s = k, (1, 6, 11, 15)[k]
        U = base.copy()
        U[mu, s][:, col] = 0.0
        lat = gpu_lattice(gpu, nc, L, dtype, field=U)
        np.testing.assert_allclose(to_np(lat.unitarity()), [1.0, 1.0], rtol=1e-5 if dtype == "f32" else 1e-13)
        np.testing.assert_allclose(O.unitarity(U, nc, L), [1.0, 1.0], rtol=1e-13)
        rep = to_np(lat.reunitarize(report=True))
        np.testing.assert_allclose(rep, [1.0, 1.0], rtol=1e-5 if dtype == "f32" else 1e-13, err_msg=what)
        got, ref = to_np(lat.export()), want.copy()
        got[mu, s] = ref[mu, s] = 0.0
        assert np.array_equal(got, ref), what

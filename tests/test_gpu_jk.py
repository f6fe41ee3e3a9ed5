"""GPU parity of the HIP J/K path against the CPU oracle (run with -m gpu).

Every case compares the library's device results element by element with
the oracle's literal sums on the same seeded inputs.  FP64 tolerance:
1e-10 absolute on J/K elements (the workload definition's bar) when screening
is off; with the production threshold tau = 1e-10 the dropped quartets are
each bounded by G_ab G_cd D_max < tau, and the test bound is stated where used.
"""
import numpy as np
import pytest

import oracle
from oracle.scf import core_guess, orthogonalizer
from synth import workloads as wl
from test_oracle import _rand_sys, _sys

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a visible GPU"
    return t


@pytest.fixture(scope="module")
def fk(torch):
    import paper_2407_21445_amd as m
    return m


def _rand_D(n, seed, nocc=None):
    rng = np.random.default_rng(seed)
    C = rng.normal(scale=0.4, size=(n, nocc or max(1, n // 3)))
    return 2.0 * C @ C.T


def _core_D(s):
    S, T, V = oracle.oneel(s)
    return core_guess(T + V, orthogonalizer(S), s["nelec"] // 2)


def _gpu_jk(fk, torch, s, D, tau, **kw):
    c = fk.FockJK(0).set_system(s).build_quartets(tau=tau, **kw)
    Dd = torch.tensor(D, dtype=torch.float64, device="cuda")
    J, K = c.build_jk(Dd, sync=True)
    return J.cpu().numpy(), K.cpu().numpy(), c


def test_device_eri_every_class_and_orientation(fk, torch):
    """Raw (ab|cd) from the production device code for every combination of
    shell angular momenta (la, lb, lc, ld) in 0..3, any orientation."""
    s = _rand_sys(31, lmax=3, natom=4, kmax=2)
    c = fk.FockJK(0).set_system(s).build_quartets(tau=0.0)
    rng = np.random.default_rng(8)
    qs = []
    for la in range(4):
        for lb in range(4):
            for lc in range(4):
                for ld in range(4):
                    at = rng.integers(0, 4, size=4)
                    qs.append([4 * at[0] + la, 4 * at[1] + lb, 4 * at[2] + lc, 4 * at[3] + ld])
    qs.append([5, 5, 5, 5])
    qs.append([15, 15, 3, 3])
    dev = c.debug_eri(qs, on_device=True)
    host = c.debug_eri(qs, on_device=False)
    for q, a, h in zip(qs, dev, host):
        b = oracle.eri_quartet(s, *q)
        scale = max(1.0, float(np.max(np.abs(b))))
        assert np.max(np.abs(a - b)) <= 1e-12 * scale, q
        assert np.max(np.abs(a - h)) <= 1e-13 * scale, q


@pytest.mark.parametrize("k", [1, 2, 3, 9])
def test_device_eri_contraction_depths(fk, torch, k):
    """Raw (ab|cd) on the device with k primitives in every shell: the ket's
    1, 4, 9 or 81 primitive pairs (an odd count ends with a single one) are
    read ahead and, for s and p shells, taken two at a time.  Same bounds as
    for every class above: the oracle within 1e-12 and the same code on the
    host within 1e-13 of max(1, |ERI|max)."""
    rng = np.random.default_rng(50 + k)
    shells = [{"atom": a, "l": l, "exps": list(rng.uniform(0.2, 3.0, size=k)), "coefs": list(rng.uniform(0.3, 1.0, size=k))}
              for a in range(2) for l in range(3)]
    s = _sys(rng.uniform(-1.5, 1.5, size=(2, 3)), shells)
    c = fk.FockJK(0).set_system(s).build_quartets(tau=0.0)
    qs = [[0, 0, 0, 0], [3, 0, 3, 0], [1, 0, 3, 0], [1, 3, 4, 0], [4, 1, 4, 1], [2, 0, 3, 0], [2, 4, 5, 1]]
    dev, host = c.debug_eri(qs, on_device=True), c.debug_eri(qs, on_device=False)
    for q, a, h in zip(qs, dev, host):
        b = oracle.eri_quartet(s, *q)
        scale = max(1.0, float(np.max(np.abs(b))))
        assert np.max(np.abs(a - b)) <= 1e-12 * scale, q
        assert np.max(np.abs(a - h)) <= 1e-13 * scale, q


def _hgp_everywhere(fk, c):
    """Selects the HGP engine for every class it is built for; returns their number."""
    n = 0
    for la in range(4):
        for lb in range(la + 1):
            for lc in range(4):
                for ld in range(lc + 1):
                    if (la, lb) < (lc, ld):
                        continue
                    try:
                        c.set_class_engine(la, lb, lc, ld, "hgp")
                        n += 1
                    except fk.FockJKError as e:
                        assert e.code == fk.FK_ERR_UNSUPPORTED
    return n


def test_device_hgp_every_class(fk, torch):
    """Raw (ab|cd) from the HGP engine's device code for every ordered
    (la, lb, lc, ld) with L <= 4 it is built for, three primitives per shell:
    against the oracle within 1e-12 (relative to max(1, |ERI|max)) and the
    same code on the host within 1e-13."""
    s = _rand_sys(31, lmax=3, natom=4, kmax=3)
    c = fk.FockJK(0).set_system(s).build_quartets(tau=0.0)
    rng = np.random.default_rng(9)
    qs = []
    for la in range(4):
        for lb in range(4):
            for lc in range(4):
                for ld in range(4):
                    n = [(l + 1) * (l + 2) // 2 for l in (la, lb, lc, ld)]
                    if la + lb + lc + ld <= 4 and n[0] * n[1] * n[2] * n[3] <= 54:
                        at = rng.integers(0, 4, size=4)
                        qs.append([4 * at[0] + la, 4 * at[1] + lb, 4 * at[2] + lc, 4 * at[3] + ld])
    assert len(qs) == 65
    dev = c.debug_eri(qs, on_device=True, engine="hgp")
    host = c.debug_eri(qs, on_device=False, engine="hgp")
    for q, a, h in zip(qs, dev, host):
        b = oracle.eri_quartet(s, *q)
        scale = max(1.0, float(np.max(np.abs(b))))
        assert np.max(np.abs(a - b)) <= 1e-12 * scale, q
        assert np.max(np.abs(a - h)) <= 1e-13 * scale, q


def test_jk_hgp_engine_spdf(fk, torch):
    """J/K with the HGP engine on every class it is built for (the Rys engine
    on the rest), unscreened, on the all-class spdf system with a random
    density: equal to the oracle within 1e-10 (relative to max(1, |J|max));
    the statistics name the engine of each launch."""
    s = _rand_sys(33, lmax=3, natom=3, kmax=2)
    s["charge"] = 1
    D = _rand_D(s["nbf"], 6)
    c = fk.FockJK(0).set_system(s)
    nh = _hgp_everywhere(fk, c)
    assert nh == 15
    c.build_quartets(tau=0.0)
    Dd = torch.tensor(D, dtype=torch.float64, device="cuda")
    J, K = c.build_jk(Dd, sync=True)
    Jo, Ko = oracle.jk(s, D)
    scale = max(1.0, float(np.max(np.abs(Jo))))
    assert np.max(np.abs(J.cpu().numpy() - Jo)) <= 1e-10 * scale
    assert np.max(np.abs(K.cpu().numpy() - Ko)) <= 1e-10 * scale
    st = c.stats()
    assert sum(1 for x in st["classes"] if x["engine"] == fk.ENGINE_HGP) == nh
    assert st["quartets"] == c.info()["nquartet_schwarz"]


def test_jk_hgp_engine_water64(fk, torch, c3):
    """(H2O)64 cc-pVDZ-type at the production threshold (tau = 1e-10,
    primitive pairs pruned at 1e-12) with the HGP engine on every class it is
    built for: sampled J/K blocks within 1e-8 of the oracle, and the same
    quartets as the all-Rys build."""
    s, D, jp, kp, Jb, Kb = c3
    c = fk.FockJK(0).set_system(s)
    _hgp_everywhere(fk, c)
    c.build_quartets(tau=1e-10, tau_prim=1e-12)
    Dd = torch.tensor(D, dtype=torch.float64, device="cuda")
    J, K = c.build_jk(Dd, sync=True)
    J, K = J.cpu().numpy(), K.cpu().numpy()
    off = oracle.bf_offsets(s)
    for (a, b), blk in zip(jp, Jb):
        assert np.max(np.abs(J[off[a]:off[a + 1], off[b]:off[b + 1]] - blk)) <= 1e-8, (a, b)
    for (a, cc), blk in zip(kp, Kb):
        assert np.max(np.abs(K[off[a]:off[a + 1], off[cc]:off[cc + 1]] - blk)) <= 1e-8, (a, cc)
    nq = c.stats()["quartets"]
    c.close()
    J2, K2, c2_ = _gpu_jk(fk, torch, s, D, tau=1e-10, tau_prim=1e-12)
    assert c2_.stats()["quartets"] == nq
    assert np.max(np.abs(J - J2)) <= 1e-11 and np.max(np.abs(K - K2)) <= 1e-11
    c2_.close()


@pytest.mark.parametrize("dens", ["core", "random"])
def test_jk_water4_unscreened(fk, torch, dens):
    s = wl.water4_sto3g()
    D = _core_D(s) if dens == "core" else _rand_D(s["nbf"], 5)
    J, K, c = _gpu_jk(fk, torch, s, D, tau=0.0)
    Jo, Ko = oracle.jk(s, D)
    assert np.max(np.abs(J - Jo)) <= 1e-10
    assert np.max(np.abs(K - Ko)) <= 1e-10
    st = c.stats()
    assert st["quartets"] == c.info()["nquartet_schwarz"] == 22155


def test_jk_water4_screened(fk, torch):
    s = wl.water4_sto3g()
    D = _core_D(s)
    J, K, c = _gpu_jk(fk, torch, s, D, tau=1e-10)
    Jo, Ko = oracle.jk(s, D)
    assert np.max(np.abs(J - Jo)) <= 1e-9
    assert np.max(np.abs(K - Ko)) <= 1e-9


def test_jk_spdf_system_unscreened(fk, torch):
    """All 55 quartet classes present; random density."""
    s = _rand_sys(33, lmax=3, natom=3, kmax=2)
    s["charge"] = 1
    D = _rand_D(s["nbf"], 6)
    J, K, c = _gpu_jk(fk, torch, s, D, tau=0.0)
    Jo, Ko = oracle.jk(s, D)
    scale = max(1.0, float(np.max(np.abs(Jo))))
    assert np.max(np.abs(J - Jo)) <= 1e-10 * scale
    assert np.max(np.abs(K - Ko)) <= 1e-10 * scale
    assert c.info()["nquartet_class"] == 55


@pytest.fixture(scope="module")
def c2():
    s = wl.c20h42_631gs()
    return s, _core_D(s)


def _blocks(s, seed, n=6):
    rng = np.random.default_rng(seed)
    l = s["sh_l"]
    dsh = [i for i in range(s["nshell"]) if l[i] == 2]
    psh = [i for i in range(s["nshell"]) if l[i] == 1]
    pairs = [(dsh[0], dsh[-1]), (dsh[3], psh[5]), (0, 1)]
    while len(pairs) < n:
        pairs.append(tuple(int(x) for x in rng.integers(0, s["nshell"], size=2)))
    return pairs


@pytest.mark.parametrize("tau,tau_prim", [(0.0, 0.0), (1e-10, 0.0), (1e-10, 1e-12)])
def test_jk_c20h42_sampled_blocks(fk, torch, c2, tau, tau_prim):
    """C20H42 6-31G*-type (384 functions), full size, core-Hamiltonian density,
    unscreened and in the configuration the benchmark times (tau = 1e-10 with
    the density screen, primitive pairs pruned at 1e-12); sampled shell blocks
    of J and K against the oracle's literal (unscreened) sums."""
    s, D = c2
    J, K, c = _gpu_jk(fk, torch, s, D, tau=tau, tau_prim=tau_prim)
    assert np.allclose(J, J.T, atol=1e-13) and np.allclose(K, K.T, atol=1e-13)
    off = oracle.bf_offsets(s)
    jp = _blocks(s, 1)
    kp = _blocks(s, 2)
    Jb, Kb = oracle.jk_blocks(s, D, jp, kp)
    tol = 1e-10 if tau == 0 else 1e-8
    for (a, b), blk in zip(jp, Jb):
        assert np.max(np.abs(J[off[a]:off[a + 1], off[b]:off[b + 1]] - blk)) <= tol, (a, b)
    for (a, cc), blk in zip(kp, Kb):
        assert np.max(np.abs(K[off[a]:off[a + 1], off[cc]:off[cc + 1]] - blk)) <= tol, (a, cc)


def test_block_tasks_of_bra_outer_classes(fk, torch, c2):
    """C20H42 unscreened with block tasks for every bra-outer lane class that
    takes them (eight-wave workgroups, the bra block lowered until the K rows
    fit): sampled blocks of J and K equal the oracle's within 1e-10."""
    s, D = c2
    wide = [(1, 0, 1, 0), (1, 1, 0, 0), (1, 1, 1, 0), (2, 0, 0, 0), (2, 0, 1, 0), (2, 1, 0, 0), (2, 1, 1, 0)]
    c = fk.FockJK(0).set_system(s)
    for w in wide:
        c.set_class_block_tasks(*w, True).set_class_engine(*w, "rys")
    c.build_quartets(tau=0.0)
    st = {x["class"]: x for x in c.stats()["classes"]}
    assert sum(st[w]["block_tasks"] > 0 and st[w]["waves_per_group"] == 8 for w in wide if w in st) >= 5
    J, K = c.build_jk(torch.tensor(D, device="cuda:0"), sync=True)
    J, K = J.cpu().numpy(), K.cpu().numpy()
    off = oracle.bf_offsets(s)
    jp, kp = _blocks(s, 5), _blocks(s, 6)
    Jb, Kb = oracle.jk_blocks(s, D, jp, kp)
    for (a, b), blk in zip(jp, Jb):
        assert np.max(np.abs(J[off[a]:off[a + 1], off[b]:off[b + 1]] - blk)) <= 1e-10, (a, b)
    for (a, cc), blk in zip(kp, Kb):
        assert np.max(np.abs(K[off[a]:off[a + 1], off[cc]:off[cc + 1]] - blk)) <= 1e-10, (a, cc)


def test_block_tasks_on_and_off(fk, torch, c2):
    """C20H42 unscreened, with and without block tasks (the (ps|ss) workgroups
    summing X_K[b_j, x], X_K[a, x] and X_J[a, b_j] of a bra block in LDS):
    both agree with the oracle's sampled blocks within 1e-10 and with each
    other (summation order only) within 1e-12."""
    s, D = c2
    res = {}
    for bt in (True, False):
        J, K, c = _gpu_jk(fk, torch, s, D, tau=0.0, block_tasks=bt)
        st = {x["class"]: x["block_tasks"] for x in c.stats()["classes"]}
        assert (st[(1, 0, 0, 0)] > 0) == bt
        res[bt] = (J, K)
        off = oracle.bf_offsets(s)
        jp, kp = _blocks(s, 3), _blocks(s, 4)
        Jb, Kb = oracle.jk_blocks(s, D, jp, kp)
        for (a, b), blk in zip(jp, Jb):
            assert np.max(np.abs(J[off[a]:off[a + 1], off[b]:off[b + 1]] - blk)) <= 1e-10, (bt, a, b)
        for (a, cc), blk in zip(kp, Kb):
            assert np.max(np.abs(K[off[a]:off[a + 1], off[cc]:off[cc + 1]] - blk)) <= 1e-10, (bt, a, cc)
    assert np.max(np.abs(res[True][0] - res[False][0])) <= 1e-12
    assert np.max(np.abs(res[True][1] - res[False][1])) <= 1e-12


def test_team_alternative_of_lane_classes(fk, torch):
    """Every lane class with a team alternative ((pp|ps), (ds|ps), (ds|pp),
    (ds|ds), (dp|ss), (dp|ps), (dd|ss), (fs|ps), (fp|ss)) switched to it:
    unscreened J and K of an s-f system still equal the oracle within 1e-10."""
    s = _rand_sys(41, lmax=3, natom=4, kmax=2)
    D = _rand_D(s["nbf"], 5)
    alts = [((1, 1, 1, 0), 3), ((2, 0, 1, 0), 6), ((2, 0, 1, 1), 6), ((2, 0, 2, 0), 6), ((2, 1, 0, 0), 6),
            ((2, 1, 1, 0), 6), ((2, 2, 0, 0), 6), ((3, 0, 1, 0), 10), ((3, 1, 0, 0), 10)]
    c = fk.FockJK(0).set_system(s)
    for cls, lanes in alts:
        c.set_class_lanes(*cls, lanes)
    c.build_quartets(tau=0.0)
    st = {x["class"]: x["team_size"] for x in c.stats()["classes"]}
    assert all(st[cls] == lanes for cls, lanes in alts if cls in st)
    assert sum(cls in st for cls, _ in alts) >= 8
    J, K = c.build_jk(torch.tensor(D, device="cuda:0"), sync=True)
    Jo, Ko = oracle.jk(s, D)
    assert np.max(np.abs(J.cpu().numpy() - Jo)) <= 1e-10
    assert np.max(np.abs(K.cpu().numpy() - Ko)) <= 1e-10


@pytest.fixture(scope="module")
def c3():
    """(H2O)64 cc-pVDZ-type at full size with a seeded dense density of
    realistic magnitude (|D| up to about 0.5; the core-Hamiltonian guess
    would need the oracle's one-electron integrals over 768 shells, minutes of
    CPU), and oracle J/K shell blocks: d-p and s-s (O and H of one molecule)
    of J, p-d and s-d (two molecules) of K."""
    s = wl.water64_ccpvdz()
    n = s["nbf"]
    C = np.random.default_rng(64).normal(scale=0.02, size=(n, n // 3))
    D = 2.0 * C @ C.T
    jp, kp = [(5, 8), (2, 6)], [(8, 5), (2, 305)]
    Jb, Kb = oracle.jk_blocks(s, D, jp, kp)
    return s, D, jp, kp, Jb, Kb


@pytest.mark.parametrize("tau,tau_prim,tol", [(1e-14, 0.0, 1e-10), (1e-10, 1e-12, 1e-8)])
def test_jk_water64_sampled_blocks(fk, torch, c3, tau, tau_prim, tol):
    """(H2O)64 cc-pVDZ-type (1600 functions), full size: sampled shell blocks
    of J and K against the oracle's literal sums, nearly unscreened (each
    dropped quartet below 1e-14) and in the configuration the benchmark times
    (tau = 1e-10, primitive pairs pruned at 1e-12, bound as for C20H42).
    Tolerances are absolute: 1e-10 on J/K elements nearly unscreened (the
    FP64 bar), 1e-8 at the production threshold."""
    s, D, jp, kp, Jb, Kb = c3
    J, K, c = _gpu_jk(fk, torch, s, D, tau=tau, tau_prim=tau_prim)
    off = oracle.bf_offsets(s)
    for (a, b), blk in zip(jp, Jb):
        err = np.max(np.abs(J[off[a]:off[a + 1], off[b]:off[b + 1]] - blk))
        print(f"water64 tau={tau:g} J[{a},{b}] max {np.max(np.abs(blk)):.2e} err {err:.2e}", flush=True)
        assert err <= tol, (a, b)
    for (a, cc), blk in zip(kp, Kb):
        err = np.max(np.abs(K[off[a]:off[a + 1], off[cc]:off[cc + 1]] - blk))
        print(f"water64 tau={tau:g} K[{a},{cc}] max {np.max(np.abs(blk)):.2e} err {err:.2e}", flush=True)
        assert err <= tol, (a, cc)
    c.close()


def test_precision_split_water64(fk, torch, c3):
    """(H2O)64 cc-pVDZ-type with the precision split at tau_fp32 = 1e-5 (the
    mixed-precision configuration, tau = 1e-10, primitive pairs pruned at
    1e-12): sampled J/K blocks against the oracle's literal sums within 1e-7,
    and the one-build energy functional 1/2 D.J - 1/4 D.K within 1e-6 Eh of
    the FP64 build on the same lists (the mixed-precision gate)."""
    s, D, jp, kp, Jb, Kb = c3
    J, K, c = _gpu_jk(fk, torch, s, D, tau=1e-10, tau_prim=1e-12, tau_fp32=1e-5)
    st = c.stats()
    n32 = sum(x["quartets"] for x in st["classes"] if x["precision"] == 32)
    assert n32 > 0
    J64, K64, c64 = _gpu_jk(fk, torch, s, D, tau=1e-10, tau_prim=1e-12)
    # every quartet computed once: the split launches together compute the FP64 build's quartets
    assert st["quartets"] == c64.stats()["quartets"]
    dE = 0.5 * np.sum(D * (J - J64)) - 0.25 * np.sum(D * (K - K64))
    print(f"water64 mixed: FP32 share {n32 / st['quartets']:.3f}, dE {dE:.2e}, "
          f"max|dJ| {np.max(np.abs(J - J64)):.2e}, max|dK| {np.max(np.abs(K - K64)):.2e}", flush=True)
    assert abs(dE) <= 1e-6
    off = oracle.bf_offsets(s)
    for (a, b), blk in zip(jp, Jb):
        assert np.max(np.abs(J[off[a]:off[a + 1], off[b]:off[b + 1]] - blk)) <= 1e-7, (a, b)
    for (a, cc), blk in zip(kp, Kb):
        assert np.max(np.abs(K[off[a]:off[a + 1], off[cc]:off[cc + 1]] - blk)) <= 1e-7, (a, cc)
    c.close()
    c64.close()


def test_edge_cases(fk, torch):
    # one atom, one s shell: a single tile holding a single quartet
    he = wl.flatten({"Z": np.array([2], dtype=np.int32), "xyz": np.zeros((1, 3)), "charge": 0, "name": "He"},
                    [{"atom": 0, "l": 0, "exps": [6.36, 1.16, 0.31], "coefs": [0.15, 0.54, 0.44]}])
    D = np.array([[2.0]])
    J, K, _ = _gpu_jk(fk, torch, he, D, tau=0.0)
    Jo, Ko = oracle.jk(he, D)
    assert abs(J[0, 0] - Jo[0, 0]) < 1e-13 and abs(K[0, 0] - Ko[0, 0]) < 1e-13
    # a threshold above every bound: nothing survives, J = K = 0 exactly
    s = wl.water4_sto3g()
    D = _core_D(s)
    J, K, c = _gpu_jk(fk, torch, s, D, tau=1e6)
    assert c.info()["nquartet_schwarz"] == 0
    assert np.all(J == 0) and np.all(K == 0)
    # repeated builds on a side stream agree (atomic ordering only)
    c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10)
    Dd = torch.tensor(D, dtype=torch.float64, device="cuda")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        J1, K1 = c.build_jk(Dd)
        J2, K2 = c.build_jk(Dd)
    side.synchronize()
    assert torch.max(torch.abs(J1 - J2)).item() < 1e-12
    assert torch.max(torch.abs(K1 - K2)).item() < 1e-12
    # host-pointer path equals the device-pointer path
    Jh, Kh = c.build_jk(D)
    assert np.max(np.abs(Jh - J1.cpu().numpy())) < 1e-12


@pytest.mark.parametrize("tau_fp32", [1e-5, 1e-3])
def test_precision_split_water4(fk, torch, tau_fp32):
    """Quartets below the split run their recurrences in FP32: every quartet
    is still computed exactly once (FP64 + FP32 counts = the unscreened
    count) and J, K and the energy functional stay within the split's error
    bound of the oracle (per quartet |(ab|cd)| < tau_fp32/2 with FP32 relative
    error; pinned here at 1e-8 in J/K and 1e-8 Eh for tau_fp32 = 1e-3)."""
    s = wl.water4_sto3g()
    D = _core_D(s)
    J, K, c = _gpu_jk(fk, torch, s, D, tau=0.0, tau_fp32=tau_fp32)
    Jo, Ko = oracle.jk(s, D)
    st = c.stats()
    n32 = sum(x["quartets"] for x in st["classes"] if x["precision"] == 32)
    n64 = sum(x["quartets"] for x in st["classes"] if x["precision"] == 64)
    assert n32 > 0 and n32 + n64 == 22155
    assert np.max(np.abs(J - Jo)) <= 1e-8 and np.max(np.abs(K - Ko)) <= 1e-8
    dE = 0.5 * np.sum(D * (J - Jo)) - 0.25 * np.sum(D * (K - Ko))
    assert abs(dE) <= 1e-8


def test_precision_split_c20h42(fk, torch, c2):
    """The benchmark configuration with the split at tau_fp32 = 1e-5: sampled
    blocks against the oracle and the one-build energy functional against the
    all-FP64 build (the mixed-precision gate is 1e-6 Eh)."""
    s, D = c2
    J, K, c = _gpu_jk(fk, torch, s, D, tau=1e-10, tau_prim=1e-12, tau_fp32=1e-5)
    J64, K64, _ = _gpu_jk(fk, torch, s, D, tau=1e-10, tau_prim=1e-12)
    st = c.stats()
    assert sum(x["quartets"] for x in st["classes"] if x["precision"] == 32) > 0
    dE = 0.5 * np.sum(D * (J - J64)) - 0.25 * np.sum(D * (K - K64))
    assert abs(dE) <= 1e-6
    assert np.max(np.abs(J - J64)) <= 1e-7 and np.max(np.abs(K - K64)) <= 1e-7
    off = oracle.bf_offsets(s)
    jp = _blocks(s, 3, n=4)
    Jb, Kb = oracle.jk_blocks(s, D, jp, jp)
    for (a, b), bj, bk in zip(jp, Jb, Kb):
        assert np.max(np.abs(J[off[a]:off[a + 1], off[b]:off[b + 1]] - bj)) <= 1e-7
        assert np.max(np.abs(K[off[a]:off[a + 1], off[b]:off[b + 1]] - bk)) <= 1e-7


def _small_batch():
    spdf = _rand_sys(33, lmax=3, natom=3, kmax=2)
    spdf["charge"] = 1
    spdf["nelec"] -= 1
    return wl.batch([wl.water4_sto3g(), wl.h2_sto3g(), wl.alkane_sys(2, "6-31gs-type"), spdf])


@pytest.mark.parametrize("tau", [0.0, 1e-10])
def test_batch_equals_single_molecules(fk, torch, tau):
    """One batched build (all molecules in the same class launches) gives
    each molecule the J and K of its own build and of the oracle."""
    b = _small_batch()
    Ds = [_rand_D(m["nbf"], 40 + i) for i, m in enumerate(b["mols"])]
    c = fk.FockJK(0).set_system(b).set_molecules(b["atom_mol"]).build_quartets(tau=tau)
    nbf, off = c.molecule_layout()
    Dd = torch.tensor(np.concatenate([d.ravel() for d in Ds]), dtype=torch.float64, device="cuda")
    J, K = c.build_jk(Dd, sync=True)
    J, K = J.cpu().numpy(), K.cpu().numpy()
    for i, (m, d) in enumerate(zip(b["mols"], Ds)):
        n = m["nbf"]
        Jb, Kb = J[off[i]:off[i + 1]].reshape(n, n), K[off[i]:off[i + 1]].reshape(n, n)
        Js, Ks, _ = _gpu_jk(fk, torch, m, d, tau=tau)
        assert np.max(np.abs(Jb - Js)) <= 1e-12 and np.max(np.abs(Kb - Ks)) <= 1e-12, i
        if tau == 0:
            Jo, Ko = oracle.jk(m, d)
            scale = max(1.0, float(np.max(np.abs(Jo))))
            assert np.max(np.abs(Jb - Jo)) <= 1e-10 * scale and np.max(np.abs(Kb - Ko)) <= 1e-10 * scale, i


def test_jk_organic_batch_sampled_blocks(fk, torch):
    """The first four molecules of the organic batch (tzvp-type, s-f, 3894
    functions) in one batched build, in the configuration the benchmark times
    (tau = 1e-10, primitive pairs pruned at 1e-12): sampled shell blocks of
    molecules 0 and 2, f-d, s-p, f-f and d-p among them, against the oracle's
    literal sums on each molecule alone, within 1e-8 relative to
    max(1, |J|max)."""
    b = wl.organic_batch(4)
    Ds = [_rand_D(m["nbf"], 80 + i) * 0.01 for i, m in enumerate(b["mols"])]
    c = fk.FockJK(0).set_system(b).set_molecules(b["atom_mol"]).build_quartets(tau=1e-10, tau_prim=1e-12)
    nbf, off = c.molecule_layout()
    Dd = torch.tensor(np.concatenate([d.ravel() for d in Ds]), dtype=torch.float64, device="cuda")
    J, K = c.build_jk(Dd, sync=True)
    J, K = J.cpu().numpy(), K.cpu().numpy()
    for i in (0, 2):
        m, n = b["mols"][i], b["mols"][i]["nbf"]
        Jm, Km = J[off[i]:off[i + 1]].reshape(n, n), K[off[i]:off[i + 1]].reshape(n, n)
        l = np.asarray(m["sh_l"])
        f = [int(x) for x in np.where(l == 3)[0]]
        d = int(np.where(l == 2)[0][0])
        p = int(np.where(l == 1)[0][0])
        jp, kp = [(f[0], d), (0, p)], [(f[0], f[-1]), (d, p)]
        Jb, Kb = oracle.jk_blocks(m, Ds[i], jp, kp)
        bo = oracle.bf_offsets(m)
        scale = max(1.0, max(float(np.max(np.abs(x))) for x in Jb))
        for (x, y), blk in zip(jp, Jb):
            err = np.max(np.abs(Jm[bo[x]:bo[x + 1], bo[y]:bo[y + 1]] - blk))
            print(f"organic mol {i} J[{x},{y}] max {np.max(np.abs(blk)):.2e} err {err:.2e}", flush=True)
            assert err <= 1e-8 * scale, (i, x, y)
        for (x, y), blk in zip(kp, Kb):
            err = np.max(np.abs(Km[bo[x]:bo[x + 1], bo[y]:bo[y + 1]] - blk))
            print(f"organic mol {i} K[{x},{y}] max {np.max(np.abs(blk)):.2e} err {err:.2e}", flush=True)
            assert err <= 1e-8 * scale, (i, x, y)
    c.close()


def test_build_in_hip_graph(fk, torch):
    """A J/K build captured in a HIP graph (no host synchronisation, no
    memset inside) and replayed several times, with eager work and
    synchronisation between replays, equals the eager build every time."""
    b = _small_batch()
    c = fk.FockJK(0).set_system(b).set_molecules(b["atom_mol"]).build_quartets(tau=1e-10)
    nmat = c.info()["nmat"]
    Dd = torch.tensor(np.concatenate([_rand_D(m["nbf"], 60 + i).ravel() for i, m in enumerate(b["mols"])]),
                      dtype=torch.float64, device="cuda")
    J0, K0 = c.build_jk(Dd, sync=True)
    J0, K0 = J0.clone(), K0.clone()
    J = torch.zeros(nmat, dtype=torch.float64, device="cuda")
    K = torch.zeros_like(J)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        c.build_jk(Dd, J, K)  # warm-up on the capture stream
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        c.build_jk(Dd, J, K)
    for rep in range(3):
        J.fill_(0.0)
        K.fill_(0.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.max(torch.abs(J - J0)).item() <= 1e-12, rep
        assert torch.max(torch.abs(K - K0)).item() <= 1e-12, rep
        c.build_jk(Dd, sync=True)  # eager work between replays


def test_autotune_keeps_results(fk, torch):
    """The autotuner only reorders work: after tuning, unscreened J/K of
    C2H6 / 6-31G*-type still equal the oracle within 1e-10, and the report
    covers every launch with positive times."""
    s = wl.alkane_sys(2, "6-31gs-type")
    S, T, V = oracle.oneel(s)
    D = core_guess(T + V, orthogonalizer(S), s["nelec"] // 2)
    c = fk.FockJK(0).set_system(s).build_quartets(tau=0.0)
    rep = c.autotune(torch.tensor(D, device="cuda:0"), reps=1)
    assert rep["configurations"] == 20 and len(rep["classes"]) == c.info()["nquartet_class"]
    assert all(r["ms_tuned"] > 0 and r["ms_default"] > 0 for r in rep["classes"])
    c.check_indices()
    J, K = c.build_jk(D)
    Jo, Ko = oracle.jk(s, D)
    assert np.max(np.abs(J - Jo)) < 1e-10 and np.max(np.abs(K - Ko)) < 1e-10


@pytest.mark.parametrize("sched", [(32, 64, 0.25), (1, 1, 1.0), (3, 17, 0.5)])
def test_extreme_schedules_keep_results(fk, torch, sched):
    """Every class under an extreme schedule (bra blocks of 1 to 32, 1 to 64
    kets per tile for the team and wave kernels, a quarter of the grid):
    unscreened J/K of C3H8 / 6-31G*-type equal the oracle within 1e-10."""
    s = wl.alkane_sys(3, "6-31gs-type")
    S, T, V = oracle.oneel(s)
    D = core_guess(T + V, orthogonalizer(S), s["nelec"] // 2)
    c = fk.FockJK(0).set_system(s)
    for la in range(3):
        for lb in range(la + 1):
            for lc in range(3):
                for ld in range(lc + 1):
                    c.set_class_schedule(la, lb, lc, ld, *sched)
    c.build_quartets(tau=0.0)
    J, K = c.build_jk(D)
    Jo, Ko = oracle.jk(s, D)
    assert np.max(np.abs(J - Jo)) < 1e-10 and np.max(np.abs(K - Ko)) < 1e-10


def test_build_progress(fk, torch):
    """A timed build without synchronisation reports its finished class
    launches until all are done; the result is the synchronous one's."""
    import time
    s = wl.alkane_sys(4, "6-31gs-type")
    S, T, V = oracle.oneel(s)
    D = torch.tensor(core_guess(T + V, orthogonalizer(S), s["nelec"] // 2), device="cuda:0")
    c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10)
    J0, K0 = c.build_jk(D, sync=True)
    J0, K0 = J0.clone(), K0.clone()
    J, K = c.build_jk(D, time_classes=True)
    t0 = time.time()
    while True:
        done, total = c.build_progress()
        assert 0 <= done <= total == c.info()["nquartet_class"]
        if done == total:
            break
        assert time.time() - t0 < 60
        time.sleep(0.001)
    torch.cuda.synchronize()
    assert float((J - J0).abs().max()) < 1e-11 and float((K - K0).abs().max()) < 1e-11


@pytest.mark.parametrize("only", ["J", "K"])
def test_j_only_and_k_only(fk, torch, c2, only):
    """FK_J_ONLY / FK_K_ONLY form one matrix and leave the other untouched.
    Unscreened on the all-class spdf system (random density) the one matrix
    equals the oracle within 1e-10 (relative to max(1, |J|max)); on C20H42 at
    tau = 1e-10, where the density screen uses only the blocks that matrix
    multiplies, sampled blocks stay within 1e-8 of the oracle and the build
    computes no more quartets than the J+K build."""
    s = _rand_sys(33, lmax=3, natom=3, kmax=2)
    s["charge"] = 1
    D = _rand_D(s["nbf"], 6)
    c = fk.FockJK(0).set_system(s).build_quartets(tau=0.0)
    Dd = torch.tensor(D, dtype=torch.float64, device="cuda")
    sentinel = torch.full_like(Dd, 7.0)
    J, K = c.build_jk(Dd, J=sentinel if only == "K" else None, K=sentinel if only == "J" else None,
                      only=only, sync=True)
    assert torch.all(sentinel == 7.0).item()
    Jo, Ko = oracle.jk(s, D)
    M, Mo = (J, Jo) if only == "J" else (K, Ko)
    assert (K if only == "J" else J) is None
    scale = max(1.0, float(np.max(np.abs(Jo))))
    assert np.max(np.abs(M.cpu().numpy() - Mo)) <= 1e-10 * scale
    # host-pointer path
    Jh, Kh = c.build_jk(D, only=only)
    Mh = Jh if only == "J" else Kh
    assert np.max(np.abs(Mh - M.cpu().numpy())) <= 1e-13 * scale
    # screened, full size
    s, D = c2
    c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10, tau_prim=1e-12)
    Dd = torch.tensor(D, dtype=torch.float64, device="cuda")
    c.build_jk(Dd, sync=True)
    nq_both = c.stats()["quartets"]
    J, K = c.build_jk(Dd, only=only, sync=True)
    assert c.stats()["quartets"] <= nq_both
    M = (J if only == "J" else K).cpu().numpy()
    off = oracle.bf_offsets(s)
    blocks = _blocks(s, 5, n=4)
    Jb, Kb = oracle.jk_blocks(s, D, blocks if only == "J" else [], blocks if only == "K" else [])
    for (a, b), blk in zip(blocks, Jb if only == "J" else Kb):
        assert np.max(np.abs(M[off[a]:off[a + 1], off[b]:off[b + 1]] - blk)) <= 1e-8, (a, b)


def test_j_engine_spd_unscreened(fk, torch):
    """The McMurchie-Davidson J engine (FK_J_ENGINE) on a random s, p, d
    system, unscreened, random density: J equals the oracle within 1e-10
    (relative to max(1, |J|max)); with K requested, K comes from the Rys
    kernels and equals the oracle too; J-only leaves K untouched."""
    s = _rand_sys(35, lmax=2, natom=4, kmax=3)
    D = _rand_D(s["nbf"], 7)
    c = fk.FockJK(0).set_system(s).build_quartets(tau=0.0)
    Dd = torch.tensor(D, dtype=torch.float64, device="cuda")
    Jo, Ko = oracle.jk(s, D)
    scale = max(1.0, float(np.max(np.abs(Jo))))
    J, K = c.build_jk(Dd, sync=True, j_engine=True)
    assert np.max(np.abs(J.cpu().numpy() - Jo)) <= 1e-10 * scale
    assert np.max(np.abs(K.cpu().numpy() - Ko)) <= 1e-10 * scale
    sentinel = torch.full_like(Dd, 7.0)
    J1, _ = c.build_jk(Dd, K=sentinel, only="J", sync=True, j_engine=True)
    assert torch.all(sentinel == 7.0).item()
    assert np.max(np.abs(J1.cpu().numpy() - Jo)) <= 1e-10 * scale


def test_j_engine_water64(fk, torch, c3):
    """(H2O)64 cc-pVDZ-type at the production threshold (tau = 1e-10,
    primitive pairs pruned at 1e-12): J from the J engine within 1e-8 of the
    oracle's sampled blocks and within 1e-8 of the Rys J everywhere."""
    s, D, jp, kp, Jb, Kb = c3
    c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10, tau_prim=1e-12)
    Dd = torch.tensor(D, dtype=torch.float64, device="cuda")
    Je, _ = c.build_jk(Dd, only="J", sync=True, j_engine=True)
    Jr, _ = c.build_jk(Dd, only="J", sync=True)
    Je, Jr = Je.cpu().numpy(), Jr.cpu().numpy()
    off = oracle.bf_offsets(s)
    for (a, b), blk in zip(jp, Jb):
        assert np.max(np.abs(Je[off[a]:off[a + 1], off[b]:off[b + 1]] - blk)) <= 1e-8, (a, b)
    assert np.max(np.abs(Je - Jr)) <= 1e-8
    c.close()


def test_j_engine_refuses_f_shells_and_batches(fk, torch):
    s = _rand_sys(33, lmax=3, natom=3, kmax=2)
    s["charge"] = 1
    c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10)
    Dd = torch.zeros((s["nbf"], s["nbf"]), dtype=torch.float64, device="cuda")
    with pytest.raises(fk.FockJKError) as e:
        c.build_jk(Dd, only="J", j_engine=True)
    assert e.value.code == fk.FK_ERR_UNSUPPORTED


def test_class_streams_join_the_callers_stream(fk, torch, c2):
    """fk_build_jk spreads the class kernels over the device's class-launch streams and
    joins them to the caller's stream: builds issued back to back on a side
    stream, with the density rescaled on that stream between them and the
    results copied on it with no synchronisation in between, equal the
    single-stream build (FK_TIME_CLASSES) of the same densities; the second
    build sees the rescaled density (J and K scale with it: Schwarz screening
    only, so the quartets do not depend on the density)."""
    s, D = c2
    c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10, tau_prim=1e-12, density_screen=False)
    Dd = torch.tensor(D, device="cuda:0")
    J0, K0 = c.build_jk(Dd.clone(), time_classes=True, sync=True)
    J0, K0 = J0.cpu().numpy(), K0.cpu().numpy()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        Dx = Dd.clone()
        J1, K1 = c.build_jk(Dx, stream=side)
        J1c, K1c = J1.clone(), K1.clone()
        Dx.mul_(0.5)
        J2, K2 = c.build_jk(Dx, stream=side)
        J2c, K2c = J2.clone(), K2.clone()
    side.synchronize()
    scale = max(1.0, float(np.abs(J0).max()), float(np.abs(K0).max()))
    for a, b in ((J1c, J0), (K1c, K0), (J2c, 0.5 * J0), (K2c, 0.5 * K0)):
        assert np.max(np.abs(a.cpu().numpy() - b)) <= 1e-12 * scale


def test_split_build_reads_its_own_density_bound(fk, torch, c2):
    """Split builds (J engine, K by the Rys kernels with the fitted-bound
    K-block skip at tau_k = 5e-6) issued back to back on one stream, the first
    on the density scaled by 1e-3, the second on the density itself: the
    second K equals that of a split build of the density alone (the same skip
    decisions; only the order of the atomics differs).  The K kernels run on
    several streams and must read the bound fitted to their own density, which
    a K-block skip with the smaller density's bound would not give."""
    s, D = c2
    Dd = torch.tensor(D, device="cuda:0")
    ca = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10, tau_prim=1e-12, tau_k=5e-6)
    Ja, Ka = ca.build_jk(Dd.clone(), j_engine=True, sync=True)
    cb = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10, tau_prim=1e-12, tau_k=5e-6)
    cb.build_jk((Dd * 1e-3).contiguous(), j_engine=True)
    Jb, Kb = cb.build_jk(Dd.clone(), j_engine=True)
    torch.cuda.synchronize()
    Ka, Kb, Ja, Jb = (x.cpu().numpy() for x in (Ka, Kb, Ja, Jb))
    scale = max(1.0, float(np.abs(Ka).max()))
    assert np.max(np.abs(Kb - Ka)) <= 1e-11 * scale
    assert np.max(np.abs(Jb - Ja)) <= 1e-11 * max(1.0, float(np.abs(Ja).max()))


@pytest.mark.parametrize("n,tau_prim", [(1, 0.0), (2, 0.0), (2, 1e-12)])
def test_cut_tiles_and_padded_groups(fk, torch, n, tau_prim):
    """Waters in the deeply contracted cc-pVDZ-type basis, unscreened: tiles
    cut over the kets' primitive pairs and kets of different primitive counts
    in one group.  J and K equal the oracle's within 1e-10 (with pruning at
    1e-12 every dropped primitive quartet is below 1e-12, at most 6561 of them
    per integral of a few largest, and the test holds 1e-9), each quartet is
    counted once and padding is not counted."""
    s = wl.water_sys(n, "ccpvdz-type")
    D = _rand_D(s["nbf"], 70 + n)
    J, K, c = _gpu_jk(fk, torch, s, D, tau=0.0, tau_prim=tau_prim)
    Jo, Ko = oracle.jk(s, D)
    tol = 1e-10 if tau_prim == 0.0 else 1e-9
    assert np.max(np.abs(J - Jo)) <= tol and np.max(np.abs(K - Ko)) <= tol
    st = c.stats()
    ns = len(s["sh_nprim"])
    npair = ns * (ns + 1) // 2
    assert st["quartets"] == npair * (npair + 1) // 2
    pp = sorted(int(s["sh_nprim"][i]) * int(s["sh_nprim"][j]) for i in range(ns) for j in range(i + 1))
    full = (sum(pp) ** 2 + sum(x * x for x in pp)) // 2
    assert st["prim_quartets"] == full if tau_prim == 0.0 else st["prim_quartets"] < full


def test_team_and_wave_kernels_with_and_without_rows(fk, torch):
    """Every class up to (ff|ff), unscreened: the team and wave kernels summing
    a bra block's K rows in LDS (the default) and adding per quartet
    (block_tasks off) both equal the oracle within 1e-10 and each other
    (summation order only) within 1e-11, as one molecule and in a batch."""
    s = _rand_sys(41, lmax=3, natom=4, kmax=2)
    D = _rand_D(s["nbf"], 77)
    Jo, Ko = oracle.jk(s, D)
    res = {}
    for bt in (True, False):
        J, K, _ = _gpu_jk(fk, torch, s, D, tau=0.0, block_tasks=bt)
        assert np.max(np.abs(J - Jo)) <= 1e-10 and np.max(np.abs(K - Ko)) <= 1e-10
        res[bt] = (J, K)
    for a, b in zip(res[True], res[False]):
        assert np.max(np.abs(a - b)) <= 1e-11
    t = _rand_sys(42, lmax=3, natom=2, kmax=3)
    E = _rand_D(t["nbf"], 78)
    c = fk.FockJK(0).set_system(wl.batch([dict(s, charge=0), dict(t, charge=0)]))
    c.set_molecules(np.repeat([0, 1], [len(s["Z"]), len(t["Z"])])).build_quartets(tau=0.0)
    J, K = c.build_jk(torch.tensor(np.concatenate([D.ravel(), E.ravel()]), device="cuda"), sync=True)
    Jt, Kt = oracle.jk(t, E)
    assert np.max(np.abs(J.cpu().numpy() - np.concatenate([Jo.ravel(), Jt.ravel()]))) <= 1e-10
    assert np.max(np.abs(K.cpu().numpy() - np.concatenate([Ko.ravel(), Kt.ravel()]))) <= 1e-10


@pytest.mark.parametrize("bra_block", [2, 4, 5, 32])
def test_bra_blocks_keep_the_screen(fk, torch, bra_block):
    """The bras of a block are screened together, four at a time: with blocks of
    any size the same quartets survive the Schwarz bound, the triangle and the
    density screen as with one bra per tile, and J and K agree within 1e-11
    (summation order only) -- J and K, K alone, and K beside the J engine with
    its K-block skip (one bra at a time)."""
    s = wl.water_sys(3, "ccpvdz-type")
    D = torch.tensor(_core_D(s), device="cuda")
    for kw, only, jeng in (({}, None, False), ({}, "K", False), ({"tau_k": 1e-6}, None, True)):
        res = []
        for bb in (1, bra_block):
            c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-8, tau_prim=0.0, bra_block=bb, **kw)
            J, K = torch.zeros_like(D), torch.zeros_like(D)
            c.build_jk(D, J, K, only=only, j_engine=jeng, sync=True)
            res.append((J.cpu().numpy(), K.cpu().numpy(), c.stats()["quartets"]))
        assert res[0][2] == res[1][2] and res[0][2] > 0
        assert np.max(np.abs(res[0][0] - res[1][0])) <= 1e-11
        assert np.max(np.abs(res[0][1] - res[1][1])) <= 1e-11


def test_contexts_with_rows_of_different_lengths(fk, torch):
    """Two live contexts whose block tasks take different amounts of LDS of the
    same kernels (C14H30 and C6H14, p and d shells): building and running the
    smaller one between two builds of the larger leaves the larger one's J and K
    as they were (summation order only, 1e-11)."""
    def ctx(n):
        s = wl.alkane_sys(n, "6-31gs-type")
        c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10, tau_prim=1e-12)
        return c, torch.tensor(_rand_D(s["nbf"], 90 + n), device="cuda")
    a, Da = ctx(14)
    J0, K0 = [x.clone() for x in a.build_jk(Da, sync=True)]
    b, Db = ctx(6)
    b.build_jk(Db, sync=True)
    J1, K1 = a.build_jk(Da, sync=True)
    scale = max(1.0, float(J0.abs().max()))
    assert float((J1 - J0).abs().max()) <= 1e-11 * scale and float((K1 - K0).abs().max()) <= 1e-11 * scale


def _split_counts(st):
    n = {(p, team): 0 for p in (32, 64) for team in (False, True)}
    for x in st["classes"]:
        n[x["precision"], x["team_size"] > 1] += x["quartets"]
    return n


@pytest.mark.parametrize("n,tau_prim", [(2, 0.0), (3, 1e-12)])
def test_cut_tiles_and_padded_groups_in_the_split(fk, torch, n, tau_prim):
    """The precision split over tiles cut along the kets' primitive pairs and
    groups of mixed primitive counts: the FP64 and the FP32 launch walk the same
    tiles and must decide alike, so that together they count every quartet once.
    An FP32 quartet is below tau_fp32 / D_max in size and errs by some 2^-19 of
    it (recurrences of a few dozen FP32 operations); it adds at most four times
    to an element, so J and K are held to 4 N tau_fp32 2^-19 for its N quartets
    (plus 1e-9 where primitive pairs are pruned) -- a lost quartet of a thousandth
    of tau_fp32 would show in the counts."""
    s = wl.water_sys(n, "ccpvdz-type")
    D = _rand_D(s["nbf"], 80 + n)
    tau32 = 1e-3
    J, K, c = _gpu_jk(fk, torch, s, D, tau=0.0, tau_prim=tau_prim, tau_fp32=tau32)
    Jo, Ko = oracle.jk(s, D)
    cnt = _split_counts(c.stats())
    ns = len(s["sh_nprim"])
    npair = ns * (ns + 1) // 2
    assert sum(cnt.values()) == npair * (npair + 1) // 2
    n32 = cnt[32, False] + cnt[32, True]
    assert n32 > 0 and cnt[64, False] > 0
    tol = 4 * n32 * tau32 * 2.0 ** -19 + 1e-9
    assert np.max(np.abs(J - Jo)) <= tol and np.max(np.abs(K - Ko)) <= tol


@pytest.mark.parametrize("block_tasks", [True, False])
def test_team_kernels_in_the_split(fk, torch, block_tasks):
    """Every class up to (ff|ff) with the precision split, the team kernels with
    and without rows in LDS, on atoms far enough apart that lane and team classes
    have quartets on both sides: counts and bounds as above."""
    s = _rand_sys(43, lmax=3, natom=4, kmax=2)
    s["xyz"] = np.asarray(s["xyz"]) * 4.0
    D = _rand_D(s["nbf"], 81)
    tau32 = 1e-4
    J, K, c = _gpu_jk(fk, torch, s, D, tau=0.0, tau_fp32=tau32, block_tasks=block_tasks)
    Jo, Ko = oracle.jk(s, D)
    cnt = _split_counts(c.stats())
    assert sum(cnt.values()) == 136 * 137 // 2 and min(cnt.values()) > 0, cnt
    tol = 4 * (cnt[32, False] + cnt[32, True]) * tau32 * 2.0 ** -19
    assert np.max(np.abs(J - Jo)) <= tol and np.max(np.abs(K - Ko)) <= tol

"""GPU tests of the initial guesses (run with -m gpu): the network kernels
(forward, backward, loss, Adam) against the FP64 oracle, the assembled and
purified learned guess against the oracle, the SAD and learned guesses inside
the SCF step, and what the trained network gains over SAD.

Tolerances: the network runs in FP32 (inputs, weights and accumulation), so
its outputs and gradients are compared relative to their largest magnitude at
1e-5 (outputs) and 1e-4 (gradients, two FP32 products deep); the purified
density inherits the prediction's FP32 error divided by the spectral gap at
the occupied/virtual boundary (about 0.03 here), hence 1e-4.
"""
import json
import math
import os

import numpy as np
import pytest

import oracle
from oracle import guess as og
from oracle.scf import run_scf as oracle_scf
from synth import geometry as geom
from synth import workloads as wl

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a visible GPU"
    return t


@pytest.fixture(scope="module")
def fk(torch):
    import paper_2407_21445_amd as m
    return m


def _rand_mlp(seed, dims, scale=1.0):
    rng = np.random.default_rng(seed)
    Ws = [scale * rng.normal(size=(dims[k], dims[k + 1])) / math.sqrt(dims[k]) for k in range(len(dims) - 1)]
    bs = [0.1 * rng.normal(size=dims[k + 1]) for k in range(len(dims) - 1)]
    # the library holds FP32 weights; the oracle gets the same rounded values
    return [W.astype(np.float32) for W in Ws], [b.astype(np.float32) for b in bs]


def _to(torch, arrs):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrs]


@pytest.mark.parametrize("n", [1, 130, 333])
def test_mlp_forward_backward_match_oracle(fk, torch, n):
    """n spans a partial tile, two tiles plus a ragged tail, and six tiles."""
    dims = [32, 64, 48, 225]
    Ws, bs = _rand_mlp(11, dims)
    rng = np.random.default_rng(12)
    X = rng.normal(size=(n, 32)).astype(np.float32)
    T = rng.normal(size=(n, 225)).astype(np.float32)
    shp = rng.choice([15 * 256 + 15, 15 * 256 + 2, 2 * 256 + 15, 2 * 256 + 2, 1 * 256 + 1], size=n).astype(np.int32)
    shapes = [(int(v) >> 8, int(v) & 255) for v in shp]
    cnt = float(sum(a * b for a, b in shapes))
    Wd, bd = _to(torch, Ws), _to(torch, bs)
    Xd, Td, Sd = _to(torch, [X, T, shp])
    work = fk.mlp_work(Wd, n)
    Y = fk.mlp_forward(Wd, bd, Xd, work)
    dY = torch.empty_like(Y)
    part, loss = fk.mse_scratch(Y.device), torch.zeros(1, dtype=torch.float64, device=Y.device)
    fk.block_mse(Y, Td, Sd, cnt, dY, part, loss)
    gW = [torch.zeros_like(W) for W in Wd]
    gb = [torch.zeros_like(b) for b in bd]
    fk.mlp_backward(Wd, bd, Xd, work, dY, gW, gb)
    torch.cuda.synchronize()
    W64, b64 = [W.astype(float) for W in Ws], [b.astype(float) for b in bs]
    Yo, pre = og.mlp_forward(W64, b64, X.astype(float))
    lo, dYo = og.block_mse(Yo, T.astype(float), shapes)
    dWo, dbo = og.mlp_backward(W64, b64, X.astype(float), pre, dYo)
    Yg = Y.cpu().numpy()
    assert np.max(np.abs(Yg - Yo)) <= 1e-5 * np.max(np.abs(Yo))
    assert float(loss.item()) == pytest.approx(lo, rel=1e-5)
    for k in range(3):
        assert np.max(np.abs(gW[k].cpu().numpy() - dWo[k])) <= 1e-4 * np.max(np.abs(dWo[k]))
        assert np.max(np.abs(gb[k].cpu().numpy() - dbo[k])) <= 1e-4 * np.max(np.abs(dbo[k]))


def test_adam_matches_oracle(fk, torch):
    dims = [32, 40, 225]
    Ws, bs = _rand_mlp(3, dims)
    rng = np.random.default_rng(4)
    gs = [rng.normal(size=W.shape).astype(np.float32) for W in Ws]
    gbs = [rng.normal(size=b.shape).astype(np.float32) for b in bs]
    Wd, bd, gWd, gbd = _to(torch, Ws), _to(torch, bs), _to(torch, gs), _to(torch, gbs)
    m1W, m1b = [torch.zeros_like(W) for W in Wd], [torch.zeros_like(b) for b in bd]
    m2W, m2b = [torch.zeros_like(W) for W in Wd], [torch.zeros_like(b) for b in bd]
    for step in (1, 2, 3):
        fk.mlp_adam(Wd, bd, gWd, gbd, m1W, m1b, m2W, m2b, step, 1e-2)
    torch.cuda.synchronize()
    for k in range(2):
        for got, w0, g in ((Wd[k], Ws[k], gs[k]), (bd[k], bs[k], gbs[k])):
            W, m, v = w0.astype(float), np.zeros(w0.shape), np.zeros(w0.shape)
            for step in (1, 2, 3):
                W, m, v = og.adam(W, g.astype(float), m, v, step, 1e-2)
            assert np.max(np.abs(got.cpu().numpy() - W)) < 1e-6


def _water2():
    return wl.make_system(geom.water_cluster(2, 8), "6-31gs-type")


def test_guess_predict_and_purify_match_oracle(fk):
    """Random seeded weights: the assembled prediction (network, bond-frame
    rotation, scatter) and the purified guess against the oracle."""
    s = _water2()
    Ws, bs = _rand_mlp(0, [192, 256, 256, 225])
    c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10)
    c.set_guess_model(Ws, bs)
    D = c.guess_predict()
    pairs = og.pair_list(s)
    X = og.features(s, pairs).astype(np.float32).astype(float)
    Do = og.assemble(s, pairs, og.mlp_forward([W.astype(float) for W in Ws], [b.astype(float) for b in bs], X)[0])
    assert np.max(np.abs(D - Do)) <= 1e-5 * np.max(np.abs(Do))
    r = c.run_scf(max_iter=0, guess=fk.GUESS_LEARNED)
    assert r["guess_used"] == fk.GUESS_LEARNED and r["iterations"] == 0
    S = oracle.oneel(s)[0]
    D0o = og.purify(S, Do, s["nelec"] // 2)
    assert np.max(np.abs(r["D"] - D0o)) < 1e-4
    assert abs(np.trace(r["D"] @ S) - s["nelec"]) < 1e-8
    DS = r["D"] @ S
    assert np.max(np.abs(DS @ DS - 2 * DS)) < 1e-8


def test_sad_guess_in_scf(fk):
    """SCF from SAD reaches the oracle's energy (1e-8 Eh) and starts from the
    oracle's SAD density."""
    s = wl.alkane_sys(2, "6-31gs-type")
    c = fk.FockJK(0).set_system(s).build_quartets(tau=0.0)
    r0 = c.run_scf(max_iter=0, guess=fk.GUESS_SAD)
    assert r0["guess_used"] == fk.GUESS_SAD
    assert np.max(np.abs(r0["D"] - og.sad_density(s))) < 1e-9
    r = c.run_scf(guess=fk.GUESS_SAD)
    assert r["converged"] and r["guess_used"] == fk.GUESS_SAD
    assert abs(r["energy"] - oracle_scf(s)["E"]) <= 1e-8


def test_learned_guess_falls_back(fk):
    """No model: the learned request runs from SAD; an element outside H, C, N,
    O would do the same (checked on the host)."""
    s = wl.water4_sto3g()
    c = fk.FockJK(0).set_system(s).build_quartets(tau=0.0)
    r = c.run_scf(guess=fk.GUESS_LEARNED)
    assert r["guess_used"] == fk.GUESS_SAD and r["converged"]
    assert abs(r["energy"] - oracle_scf(s)["E"]) <= 1e-8


def test_training_kernels_reduce_loss(fk, torch):
    """A few hundred library Adam steps on the pair blocks of two small
    converged molecules cut the masked loss by an order of magnitude."""
    from paper_2407_21445_amd import guess_train as gt
    data = {}
    for i, s in enumerate([wl.make_system(geom.alkane(4, 1, jitter=0.05), "6-31gs-type"),
                           wl.make_system(geom.water_cluster(3, 2, jitter=0.05), "6-31gs-type")]):
        c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10)
        r = c.run_scf(guess=fk.GUESS_SAD)
        assert r["converged"]
        X, sh = c.guess_pairs()
        data[i] = (X, sh, c.guess_targets(r["D"]), r["iterations"])
    data[2] = data[0]  # validation split takes one geometry
    Ws, bs, hist = gt.train(data, epochs=400, budget_s=60, batch=64, lr=3e-3, val_frac=0.3)
    first, last = hist[0][1], hist[-1][1]
    assert last < 0.1 * first, hist[:3] + hist[-3:]


MODEL = os.path.join(os.path.dirname(HERE), "paper_2407_21445_amd", "guess_631gs.npz")


@pytest.mark.skipif(not os.path.exists(MODEL), reason="no trained guess weights in the package")
def test_trained_guess_beats_sad_on_held_out(fk):
    """The first 24 held-out geometries of the guess set (never trained on;
    alkanes and water clusters, 80-532 functions): the learned guess needs
    no more SCF iterations than SAD on any of them, fewer on average, and
    never changes the converged energy by more than 1e-8 Eh."""
    from paper_2407_21445_amd import guess_train as gt
    Ws, bs = gt.load_model(MODEL)
    first = wl.GUESS_SET_SIZE - wl.GUESS_HELD_OUT
    its_sad, its_nn = [], []
    for i in range(first, first + 24):
        s = wl.guess_system(i)
        c = fk.FockJK(0).set_system(s).build_quartets(tau=1e-10)
        c.set_guess_model(Ws, bs)
        r0 = c.run_scf(guess=fk.GUESS_SAD)
        r1 = c.run_scf(guess=fk.GUESS_LEARNED)
        assert r0["converged"] and r1["converged"] and r1["guess_used"] == fk.GUESS_LEARNED
        assert abs(r1["energy"] - r0["energy"]) <= 1e-8
        its_sad.append(r0["iterations"])
        its_nn.append(r1["iterations"])
    assert all(x <= y for x, y in zip(its_nn, its_sad)), (its_sad, its_nn)
    assert np.mean(its_nn) < np.mean(its_sad), (its_sad, its_nn)


@pytest.mark.parametrize("n,dims", [(17, [4, 16, 33]), (16, [20, 32, 225]), (2049, [7, 45, 18]), (1000, [192, 256, 256, 225])])
def test_mlp_ragged_layers_match_oracle(fk, torch, n, dims):
    """Widths and row counts at the edges of the 16 x 32 tiles and 16-deep
    slices, aligned for four-wide loads and not.  An FP32 sum of m products
    errs by at most m 2^-24 sum|ab|; relative to the largest output that is
    below m 6e-8 sqrt(m) for these random operands, at most 6e-3 at m = 2049;
    sums are split 16 ways, and the existing bound 1e-4 holds for all."""
    Ws, bs = _rand_mlp(21, dims)
    rng = np.random.default_rng(22)
    X = rng.normal(size=(n, dims[0])).astype(np.float32)
    dY = rng.normal(size=(n, dims[-1])).astype(np.float32)
    Wd, bd = _to(torch, Ws), _to(torch, bs)
    Xd, Gd = _to(torch, [X, dY])
    work = fk.mlp_work(Wd, n)
    Y = fk.mlp_forward(Wd, bd, Xd, work)
    gW = [torch.full_like(W, 7.0) for W in Wd]
    gb = [torch.full_like(b, 7.0) for b in bd]
    fk.mlp_backward(Wd, bd, Xd, work, Gd, gW, gb)
    torch.cuda.synchronize()
    W64, b64 = [W.astype(float) for W in Ws], [b.astype(float) for b in bs]
    Yo, pre = og.mlp_forward(W64, b64, X.astype(float))
    dWo, dbo = og.mlp_backward(W64, b64, X.astype(float), pre, dY.astype(float))
    assert np.max(np.abs(Y.cpu().numpy() - Yo)) <= 1e-5 * np.max(np.abs(Yo))
    for k in range(len(dims) - 1):
        assert np.max(np.abs(gW[k].cpu().numpy() - dWo[k])) <= 1e-4 * np.max(np.abs(dWo[k]))
        assert np.max(np.abs(gb[k].cpu().numpy() - dbo[k])) <= 1e-4 * np.max(np.abs(dbo[k]))


def test_mlp_more_rows_than_one_grid_dimension(fk, torch):
    """1050011 rows are more 16-row tiles than a grid's y can count (65535, at
    1048560 rows).  Small layers against the same sums in FP64 on the device: an
    output is a sum of at most 8 products (errors below 8 2^-23 of sum |ab|), a
    weight gradient a sum over the rows, whose FP32 parts of n / 16 random terms
    err by about 2^-24 sqrt(n) of its own size; held to 1e-5 and, as above, 1e-4
    of the largest value."""
    n, dims = 1050011, [3, 8, 5]
    Ws, bs = _rand_mlp(23, dims)
    Wd, bd = _to(torch, Ws), _to(torch, bs)
    g = torch.Generator(device="cuda").manual_seed(24)
    X = torch.randn(n, dims[0], device="cuda", generator=g)
    dY = torch.randn(n, dims[-1], device="cuda", generator=g) + 0.5
    work = fk.mlp_work(Wd, n)
    Y = fk.mlp_forward(Wd, bd, X, work)
    W64 = [w.double().requires_grad_() for w in Wd]
    b64 = [v.double().requires_grad_() for v in bd]
    Yo = torch.nn.functional.silu(X.double() @ W64[0] + b64[0]) @ W64[1] + b64[1]
    assert float((Y - Yo.detach()).abs().max()) <= 1e-5 * float(Yo.detach().abs().max())
    (Yo * dY.double()).sum().backward()
    gW = [torch.full_like(W, 7.0) for W in Wd]
    gb = [torch.full_like(b, 7.0) for b in bd]
    fk.mlp_backward(Wd, bd, X, work, dY, gW, gb)
    for got, want in zip(gW + gb, W64 + b64):
        assert float((got - want.grad).abs().max()) <= 1e-4 * float(want.grad.abs().max())


@pytest.mark.parametrize("n,din,dout", [(8128, 3, 5), (8129, 17, 64), (2049, 16, 225), (2048, 37, 250), (513, 31, 1023)])
def test_mlp_forward_of_many_rows_is_the_same_chain(fk, torch, n, din, dout):
    """From 128 tiles of 64 x 64 outputs on the forward layer stages slabs in LDS
    (8128 rows of one column of tiles are 127: the last without).  Every output is
    the same chain of products added in the order of k as in a call with few rows,
    so the two agree bit for bit, on ragged rows, columns and depths; and a sum of
    din products errs by less than din 2^-24 sum |xw|, held to 1e-5 of the largest."""
    (W,), (b,) = _rand_mlp(25, [din, dout])
    Wd, bd = _to(torch, [W]), _to(torch, [b])
    X = torch.randn(n, din, device="cuda", generator=torch.Generator(device="cuda").manual_seed(26))
    Y = fk.mlp_forward(Wd, bd, X, fk.mlp_work(Wd, n))
    few = torch.cat([fk.mlp_forward(Wd, bd, x.contiguous(), fk.mlp_work(Wd, n)) for x in X.split(100)])
    assert torch.equal(Y, few)
    want = X.double() @ Wd[0].double() + bd[0].double()
    assert float((Y - want).abs().max()) <= 1e-5 * float(want.abs().max())


def test_mlp_forward_equals_a_chain_of_fused_products(fk, torch):
    """The forward layer's outputs are fma(x_k, w_k, sum) over k = 0, 1, ... with
    the bias added last, bit for bit, in either kernel (5 and 8200 rows; 19
    products, which no slice of 16 divides)."""
    import ctypes
    import ctypes.util
    fmaf = ctypes.CDLL(ctypes.util.find_library("m")).fmaf
    fmaf.argtypes, fmaf.restype = [ctypes.c_float] * 3, ctypes.c_float
    (W,), (b,) = _rand_mlp(27, [19, 7])
    Wd, bd = _to(torch, [W]), _to(torch, [b])
    X = np.random.default_rng(28).normal(size=(8200, 19)).astype(np.float32)
    for n in (5, 8200):
        Xd = torch.tensor(X[-n:], device="cuda")
        Y = fk.mlp_forward(Wd, bd, Xd, fk.mlp_work(Wd, n)).cpu().numpy()
        for r in (0, 3, n - 1):
            for c in range(7):
                s = 0.0
                for k in range(19):
                    s = fmaf(float(X[-n:][r, k]), float(W[k, c]), s)
                assert Y[r, c] == np.float32(np.float32(s) + b[c]), (n, r, c)

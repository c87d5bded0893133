"""Kernel forms of single levels against the FP64 oracle, at the grid sizes
where their tilings and branches end.

Tolerances as for the other parity tests: both sides are converged far below
the target, so FP64 solves agree to 1e-8 and FP32-refined ones to 1e-6
(relative to the deviation from the background), adjoints to 1e-8 and 1e-5.
"""
import re

import numpy as np
import pytest
import torch

import oracle
from paper_2110_00328_amd import api

pytestmark = pytest.mark.gpu

CH = oracle.C_OVER_H0
DEV = torch.device("cuda:0")
KIND = {"fr": oracle.FR, "sym": oracle.SYM, "cq": oracle.CQ}


def inputs(model, n, seed, sig=1.0, **kw):
    """oracle params, ABI params, density contrast"""
    if model == "sym":
        kw = dict(a=1.0, a_star=0.5, xi=2.0 / CH, beta_star=1.0, **kw)
    elif model == "fr":
        kw = dict(dict(fr0=1e-5), **kw)
    g = np.random.default_rng(seed).standard_normal((n, n, n))
    d = np.exp(sig * g - 0.5 * sig * sig) - 1
    box = float(n)
    return (oracle.params(KIND[model], n, box, **kw), api.model_params(box, **kw),
            (d - d.mean()).astype(np.float32))


def deviation(model, x, P):
    x = np.asarray(x, dtype=np.float64)
    if model == "cq":  # the uniform mode is nearly a null mode
        return x - x.mean()
    return x - (-1.0 if model == "fr" else 1.0) * oracle.background(P)


def rel_err(model, x, ref, P):
    a, b = deviation(model, x, P), deviation(model, ref, P)
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def solve_and_adjoint_match(model, n, prec, cycle="V", seed=71, **kw):
    P, prm, delta = inputs(model, n, seed, **kw)
    d64 = delta.astype(np.float64)
    ref, _, _, _ = oracle.solve(P, d64, tol=1e-12)
    mg = api.Context(n, device=DEV)
    dt = torch.from_numpy(delta).to(DEV)
    o = api.solver_opts(precision=prec, cycle=cycle, max_cycles=64)
    print("solve and adjoint", model, n, prec, cycle, kw, flush=True)
    field, st = mg.solve(model, prm, dt, tol=1e-11 if prec == "fp64" else 1e-9, opts=o)
    err = rel_err(model, field.cpu().numpy(), -ref if model == "fr" else ref, P)
    # adjoint at the oracle's field, right-hand side without a uniform mode
    gv = np.random.default_rng(seed + 1).standard_normal((n, n, n))
    gv -= gv.mean()
    gref, _, _ = oracle.adjoint(P, d64, ref, gv, tol=1e-12, solver="cg")
    sgn = -1.0 if model == "fr" else 1.0
    gd, sa = mg.solve_adjoint(model, prm, dt, torch.from_numpy(sgn * ref).to(DEV),
                              torch.from_numpy(sgn * gv).to(DEV),
                              tol=1e-11 if prec == "fp64" else 1e-9, opts=o)
    aerr = np.linalg.norm(gd.cpu().numpy() - gref) / np.linalg.norm(gref)
    mg.close()
    print(f"  cycles {st.vcycles} / {sa.vcycles}, field {err:.2e}, adjoint {aerr:.2e}", flush=True)
    assert err < (1e-8 if prec == "fp64" else 1e-6)
    assert aerr < (1e-8 if prec == "fp64" else 1e-5)


# 8: one cell per thread on the coarsest 4^3; 20 -> 10 and 24 -> 12 -> 6: the
# colours on different waves; 28 -> 14: a coarsest level of more cells than
# threads; 32 -> 16: two positions per thread
# (the oracle solves a coarsest 10^3 of coupled quintessence as one dense
# system, which takes minutes)
@pytest.mark.parametrize("model,n", [("fr", 8), ("fr", 20), ("fr", 24), ("fr", 28), ("fr", 32),
                                     ("sym", 20), ("sym", 28), ("sym", 32),
                                     ("cq", 16), ("cq", 24), ("cq", 32)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_small_levels_match_oracle(model, prec, n):
    solve_and_adjoint_match(model, n, prec)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_small_levels_second_visits_and_other_exponents(prec):
    solve_and_adjoint_match("sym", 32, prec, cycle="W")
    solve_and_adjoint_match("fr", 32, prec, cycle="F", fr_n=2)


# one launch per way down and way up of a level against one per operation:
# 8 and 12 (the tile's frame wraps the whole period), rows of 4 to 40 cells, 12
# and 20 (rows of no multiple of 4), 96 and 160 (levels above the limit lead
# into it), 16-bit and FP32 storage
@pytest.mark.parametrize("model,n,cycle,fp16", [
    ("fr", 8, "V", "1"), ("sym", 12, "V", "1"), ("fr", 20, "V", "1"), ("fr", 32, "W", "0"),
    ("sym", 40, "F", "1"), ("fr", 56, "V", "0"), ("sym", 64, "W", "1"), ("fr", 80, "V", "1"),
    ("fr", 96, "F", "1"), ("sym", 160, "V", "0")])
def test_one_launch_levels_are_bit_identical(monkeypatch, model, n, cycle, fp16):
    _, prm, delta = inputs(model, n, 91)
    dt = torch.from_numpy(delta).to(DEV)
    gv = torch.from_numpy(np.random.default_rng(92).standard_normal((n, n, n))).to(DEV)
    monkeypatch.setenv("MGGPU_FP16_STORAGE", fp16)
    got = []
    for limit in ("0", "80"):
        monkeypatch.setenv("MGGPU_MID_MAX_N", limit)
        mg = api.Context(n, device=DEV)
        o = api.solver_opts(cycle=cycle)
        print("one-launch levels", model, n, cycle, fp16, limit, flush=True)
        field, _ = mg.solve(model, prm, dt, tol=1e-6, opts=o)
        gd, _ = mg.solve_adjoint(model, prm, dt, field, gv, tol=1e-6, opts=o)
        got.append((field, gd))
        mg.close()
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])


# boxes solved together: the marching outer step with two master buffers (rows
# of a multiple of 8 cells, aligned arrays) against the separate kernels, which
# arrays at odd addresses take; one-launch levels bit for bit against separate
# ones.  From the background, from a given field, stopped at once (the field is
# then the start) and with two sweeps (no one-launch levels).
@pytest.mark.parametrize("sizes,cycle,nu,start,tol", [
    ((8, 16, 8), "V", 1, False, 1e-8), ((12, 24), "V", 1, False, 1e-8),
    ((32, 48, 64), "V", 1, True, 1e-8), ((32, 40), "F", 1, False, 1e-8),
    ((64, 64, 96), "W", 2, False, 1e-8), ((16, 72), "V", 1, False, 1e30),
    ((24, 32), "V", 1, True, 1e30)])
def test_boxes_together_take_the_same_steps(monkeypatch, sizes, cycle, nu, start, tol):
    got = []
    for limit, off in (("80", 0), ("0", 0), ("80", 1)):
        monkeypatch.setenv("MGGPU_MID_MAX_N", limit)
        mg = api.Context(8, device=DEV)
        mg.batched_set_config(256, 1, 2)
        boxes = []
        for q, n in enumerate(n for n in sizes for _ in range(2)):
            model = ("fr", "sym")[q % 2]
            P, prm, d = inputs(model, n, 300 + q)
            m = n ** 3
            bg = (-1.0 if model == "fr" else 1.0) * oracle.background(P)
            field = torch.full((m + 1,), 1.25 * bg, dtype=torch.float64, device=DEV)[off:off + m]
            delta = torch.zeros(m + 1, dtype=torch.float32, device=DEV)[off:off + m]
            delta.copy_(torch.from_numpy(d.ravel()))
            force = torch.zeros(3 * m + 1, dtype=torch.float32, device=DEV)[off:off + 3 * m]
            boxes.append(dict(n=n, model=model, params=prm, delta=delta.view(n, n, n),
                              field=field.view(n, n, n), force=force.view(3, n, n, n),
                              field_in=1 if start else 0, bg=bg))
        print("boxes together", sizes, cycle, nu, start, limit, off, flush=True)
        st = mg.solve_batched(boxes, tol=tol,
                              opts=api.solver_opts(cycle=cycle, nu_pre=nu, nu_post=nu))
        assert all(s.status == 0 and s.rel_resid <= tol for s in st)
        got.append([(b["field"].cpu().numpy(), b["force"].cpu().numpy(), b["bg"]) for b in boxes])
        mg.close()
    for one, sep, plain in zip(*got):
        assert np.array_equal(one[0], sep[0]) and np.array_equal(one[1], sep[1])
        if tol > 1:
            if start:
                assert np.all(one[0] == 1.25 * one[2])
            assert np.allclose(one[0], (1.25 if start else 1.0) * one[2], rtol=1e-13, atol=0.0)
            assert np.array_equal(one[0], plain[0])
            assert not one[1].any() and not plain[1].any()
            continue
        for a, b, ref in zip(one[:2], plain[:2], (one[2], 0.0)):
            assert np.linalg.norm(a - b) <= 1e-6 * np.linalg.norm(b - ref)


# particles binned by tiles of 16^3 cells against direct deposits: one thin tile,
# a thin last tile of 2 to 14 cells, particles on the last layers and the seam
@pytest.mark.parametrize("n", [10, 16, 18, 30, 34, 48, 50])
def test_binned_deposit_on_any_side_equals_direct(n, monkeypatch):
    rng = np.random.default_rng(500 + n)
    pos = rng.uniform(0, n, (40011, 3)).astype(np.float32)
    pos[:3000] = np.sort(pos[:3000], axis=0)
    for a in range(3):
        pos[3000 + 50 * a:3050 + 50 * a, a] = np.float32(n - 0.4)
        pos[3200 + 50 * a:3250 + 50 * a, a] = np.float32(0.3)
        pos[3400 + 50 * a:3450 + 50 * a, a] = np.float32(16 * ((n - 1) // 16) - 0.2)
    t = torch.from_numpy(pos).to(DEV)
    got = []
    for mode in ("0", "1"):
        monkeypatch.setenv("MGGPU_CIC_DIRECT", mode)
        mg = api.Context(n, device=DEV)
        print("binned deposit", n, mode, flush=True)
        mg.cic(t[:100].contiguous())  # the binned path's buffers grow
        got.append(mg.cic(t).cpu().numpy())
        mg.close()
    assert np.array_equal(got[0], got[1])
    ref = oracle.cic(n, pos.astype(np.float64))
    assert np.max(np.abs(got[0] - ref)) <= 1e-6 * (1 + np.max(np.abs(ref)))


# gathers at particles on the seam of each axis against CIC weights in FP64
@pytest.mark.parametrize("n", [8, 10, 18])
def test_gathers_on_the_seam(n):
    rng = np.random.default_rng(600 + n)
    pos = rng.uniform(0, n, (1003, 3)).astype(np.float32)
    for a in range(3):
        pos[100 * a:100 * a + 50, a] = np.float32(n - 0.3)
        pos[100 * a + 50:100 * a + 100, a] = np.float32(0.2)
    x = pos.astype(np.float64) - 0.5
    i0 = np.floor(x).astype(int)
    t = x - i0
    grid = rng.standard_normal((3, n, n, n)).astype(np.float32)
    want = np.zeros((len(pos), 3))
    for q in range(8):
        d = [(q >> a) & 1 for a in range(3)]
        w = np.prod([t[:, a] if d[a] else 1 - t[:, a] for a in range(3)], axis=0)
        i, j, k = [(i0[:, a] + d[a]) % n for a in range(3)]
        want += w[:, None] * grid[:, k, j, i].T
    mg = api.Context(n, device=DEV)
    tp, tg = torch.from_numpy(pos).to(DEV), torch.from_numpy(grid).to(DEV)
    print("gathers", n, flush=True)
    three = mg.interp_to_particles(tg, tp).cpu().numpy()
    mom = torch.from_numpy(rng.standard_normal(pos.shape).astype(np.float32)).to(DEV)
    fric = mg.symmetron_friction(api.model_params(float(n), a=1.0, a_star=0.5),
                                 tg[1].double(), tp, mom).cpu().numpy()
    mg.close()
    assert np.max(np.abs(three - want)) <= 2.0 ** -23 * np.max(np.abs(grid))
    # the same factor for every particle
    f = want[:, 1:2] * mom.cpu().numpy().astype(np.float64)
    c = np.sum(fric * f) / np.sum(f * f)
    assert np.max(np.abs(fric - c * f)) <= 2.0 ** -22 * np.max(np.abs(c * f))


# The level kernels that run one operation each, which levels of at most 80
# cells a side reach only without the one-launch form: marching in z against one
# plane per thread (restriction, smoother), and the prolongation formed inside
# the half-sweep (f(R) and adjoint) against the two kernels.  Bit for bit the
# same.  64^3: coarse sides 32 and 16, one tile of whole rows; 96^3: 48, 24,
# ragged last tiles; 160^3: 80, 40, 20; 3 planes leave a ragged last chunk.
MARCH = dict(MGGPU_MARCH_MIN_BLOCKS="0", MGGPU_SMOOTH_MARCH_KT="4")
PLANE = dict(MGGPU_MARCH_MIN_BLOCKS="2147483647", MGGPU_SMOOTH_MARCH_KT="0")


def same_with(monkeypatch, model, n, fp16, envs):
    _, prm, delta = inputs(model, n, 93)
    dt = torch.from_numpy(delta).to(DEV)
    gv = torch.from_numpy(np.random.default_rng(94).standard_normal((n, n, n))).to(DEV)
    monkeypatch.setenv("MGGPU_MID_MAX_N", "0")
    monkeypatch.setenv("MGGPU_FP16_STORAGE", fp16)
    got = []
    for env in envs:
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        mg = api.Context(n, device=DEV)
        print("separate level kernels", model, n, fp16, env, flush=True)
        field, _ = mg.solve(model, prm, dt, tol=1e-8)
        gd, _ = mg.solve_adjoint(model, prm, dt, field, gv, tol=1e-8)
        got.append((field, gd))
        mg.close()
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("model,n,fp16", [("fr", 64, "1"), ("sym", 64, "0"), ("fr", 96, "0"),
                                          ("sym", 96, "1"), ("fr", 160, "1")])
def test_marching_level_kernels_below_the_one_launch_limit(monkeypatch, model, n, fp16):
    monkeypatch.setenv("MGGPU_PROLONG_SMOOTH_KT", "0")
    same_with(monkeypatch, model, n, fp16, (PLANE, MARCH))


@pytest.mark.parametrize("model,n,kt,fp16", [("fr", 64, "1", "1"), ("fr", 64, "2", "0"),
                                             ("fr", 96, "4", "1"), ("fr", 96, "8", "0"),
                                             ("fr", 160, "3", "0"), ("sym", 96, "4", "1")])
def test_fused_prolongation_below_the_one_launch_limit(monkeypatch, model, n, kt, fp16):
    for k, v in MARCH.items():
        monkeypatch.setenv(k, v)
    monkeypatch.setenv("MGGPU_PROLONG_SMOOTH_MIN_BLOCKS", "0")
    same_with(monkeypatch, model, n, fp16,
              [dict(MGGPU_PROLONG_SMOOTH_KT=k) for k in ("0", kt)])


# a tuning file of a library with other kernels is not taken: the batch is tuned
# again and the entry stays beside the new one
def test_earlier_tuning_is_not_taken(monkeypatch, tmp_path):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("MGGPU_TUNE_CACHE", str(path))
    _, prm, d = inputs("fr", 16, 97)
    field = torch.empty((16, 16, 16), dtype=torch.float64, device=DEV)
    box = dict(n=16, model="fr", params=prm, delta=torch.from_numpy(d).to(DEV), field=field)

    def keys():
        print("earlier tuning", flush=True)
        mg = api.Context(16, device=DEV)
        mg.solve_batched([box], tol=1e-6)
        mg.close()
        return [line.split('"')[1] for line in path.read_text().splitlines() if '"' in line]

    (key,) = keys()
    earlier = re.sub(r"batched\d+:", "batched2:", key)
    assert earlier != key
    path.write_text('{\n  "%s": [1024, 0, 0, 0.001]\n}\n' % earlier)
    assert sorted(keys()) == sorted([earlier, key])


# boxes together without memory for the second masters and the one-launch levels'
# scratch (refused from the host): the separate kernels, which boxes at odd
# addresses take too, on every call
def test_boxes_together_in_the_smaller_pool(monkeypatch):
    got = []
    for refused, off in (("1", 0), (None, 1)):
        if refused:
            monkeypatch.setenv("MGGPU_TEST_BATCH_POOL", refused)
        else:
            monkeypatch.delenv("MGGPU_TEST_BATCH_POOL")
            monkeypatch.setenv("MGGPU_MID_MAX_N", "0")
        mg = api.Context(8, device=DEV)
        mg.batched_set_config(256, 1, 2)
        for sizes in ((32, 24), (16, 16), (32, 24, 40)):  # the pool grows, is kept, grows
            boxes = []
            for q, n in enumerate(sizes):
                model = ("fr", "sym")[q % 2]
                _, prm, d = inputs(model, n, 400 + q)
                delta = torch.zeros(n ** 3 + 1, dtype=torch.float32, device=DEV)[off:off + n ** 3]
                delta.copy_(torch.from_numpy(d.ravel()))
                boxes.append(dict(n=n, model=model, params=prm, delta=delta.view(n, n, n),
                                  field=torch.empty((n, n, n), dtype=torch.float64, device=DEV),
                                  force=torch.empty((3, n, n, n), device=DEV)))
            print("boxes in the smaller pool", sizes, refused, off, flush=True)
            st = mg.solve_batched(boxes, tol=1e-8)
            assert all(s.status == 0 and s.rel_resid <= 1e-8 for s in st)
            got.append([(b["field"], b["force"]) for b in boxes])
        mg.close()
    for small, plain in zip(got[:3], got[3:]):
        for a, b in zip(small, plain):
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])

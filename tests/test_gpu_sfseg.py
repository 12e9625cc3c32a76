"""The full SFSeg operator (Eq. 2 Taylor affinity, Eq. 5-7; alpha > 0, unary
map s = S^p distinct from the pairwise feature f) on the GPU against the FP64
oracle: one step on ragged shapes spanning several tiles at every compiled
radius (FP32 <= 1e-5 relative L2, FP64 <= 1e-12), the step's sums, the
iteration and its stopping rule, the dense Perron vector on a tiny volume,
sampled voxels at full frame size, the unary power and the affinity check."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import Kernel as OK

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {torch.float32: 1e-5, torch.float64: 1e-12}


@pytest.fixture(scope="module")
def S():
    import paper_2212_08058_amd as P
    from paper_2212_08058_amd import sfseg
    return P, sfseg


def rel_l2(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b))


def okf(k):
    return OK(float(np.float32(k.sigma_s)), float(np.float32(k.sigma_t)), k.r_s, k.r_t)


def _fields(shape, seed, p=0.2):
    """s: a soft blob mask to the power p (the unary map); f: another soft mask
    in [0, 1] (the pairwise feature, standing in for optical-flow magnitude)."""
    T, H, W = shape
    S0, _ = synth.blob_clip(T, H, W, 3, seed)
    F0, _ = synth.blob_clip(T, H, W, 2, seed + 1000)
    return (S0.astype(np.float64) ** p), F0.astype(np.float64)


CASES = [
    ((5, 37, 70), (2.0, 1.0, 4, 2), 1.0),      # ragged, one tile column
    ((9, 40, 131), (4.0, 1.5, 8, 3), 0.5),     # three tiles across
    ((12, 70, 150), (5.0, 2.0, 15, 5), 1.0),   # the largest compiled radii, two tile rows
    ((3, 17, 19), (1.3, 0.7, 1, 1), 0.8),
    ((1, 1, 1), (1.0, 1.0, 2, 1), 1.0),        # single voxel
    ((6, 33, 5), (2.0, 1.0, 0, 0), 1.0),       # no neighbours
    ((20, 16, 64), (3.0, 1.0, 16, 5), 0.3),    # radius above the frame size
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("shape,kp,alpha", CASES)
def test_sfseg_step_matches_oracle(S, shape, kp, alpha, dtype):
    P, Sf = S
    kern = P.Kernel(*kp)
    if dtype == torch.float64 and (kern.r_s > 4 or kern.r_t > 2):
        pytest.skip("the FP64 build covers radii up to (4, 2)")
    s, f = _fields(shape, 7)
    x = np.random.default_rng(8).uniform(-0.2, 1.0, shape)
    if dtype == torch.float32:
        s, f, x = (v.astype(np.float32).astype(np.float64) for v in (s, f, x))
    print(f"case: sfseg step {shape} r=({kern.r_s},{kern.r_t}) alpha {alpha} {dtype}", flush=True)
    scale = 0.6
    z, sums = Sf.sfseg_step(*(torch.from_numpy(v).to(DEV).to(dtype) for v in (s, f, x)), kern, alpha, x_scale=scale)
    torch.cuda.synchronize()
    ref = oracle.sfseg_apply(s, f, x * scale, alpha, okf(kern))
    zz = z.double().cpu().numpy()
    err = rel_l2(zz, ref)
    print(f"  rel L2 {err:.3e}")
    assert err <= TOL[dtype], err
    sm = sums.cpu().numpy()
    assert abs(sm[0] - np.sum(zz * zz)) <= 1e-12 * np.sum(zz * zz)
    assert abs(sm[1] - scale * np.sum(zz * x)) <= 1e-12 * abs(scale * np.sum(zz * x)) + 1e-300


def test_sfseg_iteration_matches_oracle(S):
    """Ten applications from the uniform start: every iterate's direction and
    lambda against the oracle's iteration."""
    P, Sf = S
    kern = P.Kernel(2.0, 1.0, 4, 2)
    s, f = _fields((8, 64, 112), 11)
    s, f = (v.astype(np.float32) for v in (s, f))
    x, r = Sf.sfseg_iterate(torch.from_numpy(s).to(DEV), torch.from_numpy(f).to(DEV), kern, 1.0, iters=10)
    torch.cuda.synchronize()
    xr, info = oracle.sfseg_iterate(s, f, 1.0, okf(kern), iters=10)
    err = rel_l2(x.double().cpu().numpy(), xr)
    print(f"sfseg 10 iterations: rel L2 {err:.3e}, lambda {r['lambda_']:.9g} vs {info.lambdas[-1]:.9g}, "
          f"residual {r['residual']:.4e} vs {info.residuals[-1]:.4e}")
    assert r["iters"] == 10 and err <= 1e-5
    assert abs(r["lambda_"] - info.lambdas[-1]) <= 1e-5 * info.lambdas[-1]
    assert abs(r["residual"] - info.residuals[-1]) <= 1e-4 * info.residuals[-1]


def test_sfseg_tolerance_run_and_start_vector(S):
    """Stop at the first residual below tol (within two iterations of the
    oracle's count), converged vector within 1e-3 cosine distance; a given
    start vector (Alg. 1 starts from the unary map) matches the oracle's
    iteration from the same start."""
    P, Sf = S
    kern = P.Kernel(2.0, 1.0, 4, 2)
    s, f = _fields((6, 40, 72), 21)
    s, f = (v.astype(np.float32) for v in (s, f))
    sd, fd = torch.from_numpy(s).to(DEV), torch.from_numpy(f).to(DEV)
    x, r = Sf.sfseg_iterate(sd, fd, kern, 1.0, tol=1e-4, max_iters=500)
    xr, info = oracle.sfseg_iterate(s, f, 1.0, okf(kern), tol=1e-4, cap=500)
    cosd = 1.0 - float(np.sum(x.double().cpu().numpy() * xr))
    print("tolerance run", r["iters"], info.iters, f"cos distance {cosd:.2e}")
    assert r["converged"] and info.converged and abs(r["iters"] - info.iters) <= 2 and cosd <= 1e-3
    x, r = Sf.sfseg_iterate(sd, fd, kern, 1.0, iters=6, x0=sd.clone())
    xr, info = oracle.sfseg_iterate(s, f, 1.0, okf(kern), x0=s, iters=6)
    assert rel_l2(x.double().cpu().numpy(), xr) <= 1e-5


def test_sfseg_dense_perron_vector(S):
    """Tiny volume, FP64: the converged GPU vector is the nonnegative principal
    eigenvector of the explicit matrix (numpy eigh)."""
    P, Sf = S
    kern = P.Kernel(2.0, 1.0, 2, 1)
    s, f = _fields((3, 8, 12), 31)
    M = oracle.sfseg_dense(s, f, 1.0, okf(kern))
    lam, v, w = oracle.perron(M)
    x, r = Sf.sfseg_iterate(torch.from_numpy(s).to(DEV), torch.from_numpy(f).to(DEV), kern, 1.0, tol=1e-12,
                            max_iters=20000)
    xf = x.cpu().numpy().reshape(-1)
    print("dense perron", r["iters"], r["lambda_"], lam, 1 - float(xf @ v))
    assert r["converged"] and 1.0 - float(xf @ v) < 1e-10
    assert abs(r["lambda_"] - lam) <= 1e-9 * lam and xf.min() >= -1e-12


def test_sfseg_full_frame_sampled(S):
    """64 x 480 x 854 at r = (15, 5), alpha = 1, p = 0.2: one step from a
    seeded start, sampled voxels against the oracle's direct loop."""
    P, Sf = S
    kern = P.Kernel(5.0, 2.0, 15, 5)
    shape = (64, 480, 854)
    s, f = _fields(shape, 41)
    s, f = (v.astype(np.float32) for v in (s, f))
    x = np.random.default_rng(42).uniform(0.0, 1.0, shape).astype(np.float32)
    print("case: sfseg full frame 64x480x854", flush=True)
    z, _ = Sf.sfseg_step(*(torch.from_numpy(v).to(DEV) for v in (s, f, x)), kern, 1.0)
    idx = np.random.default_rng(43).integers(0, s.size, 400)
    got = z.reshape(-1)[torch.from_numpy(idx).to(DEV)].double().cpu().numpy()
    ref = oracle.sfseg_apply_at(s, f, x, 1.0, okf(kern), idx)
    err = rel_l2(got, ref)
    print(f"  sampled rel L2 {err:.3e}")
    assert err <= 1e-5


def test_sfseg_unary_and_affinity_check(S):
    """s = S^p against numpy; alpha (max f - min f)^2 > 1 (some affinity of
    Eq. 2 negative) is refused by the iteration with STPI_EINVAL, flags bit 4."""
    P, Sf = S
    from paper_2212_08058_amd import _native as N
    rng = np.random.default_rng(51)
    Sv = rng.uniform(0.0, 1.0, (4, 20, 30)).astype(np.float32)
    Sv[0, 0, :3] = 0.0
    s = Sf.sfseg_unary(torch.from_numpy(Sv).to(DEV), 0.2).cpu().numpy()
    ref = Sv.astype(np.float64) ** 0.2
    assert np.max(np.abs(s - ref)) <= 2e-7 * np.max(ref) and np.all(s[0, 0, :3] == 0)
    kern = P.Kernel(2.0, 1.0, 4, 2)
    f = rng.uniform(0.0, 1.0, Sv.shape).astype(np.float32)
    sd, fd = torch.from_numpy(s).to(DEV), torch.from_numpy(f).to(DEV)
    _, r = Sf.sfseg_iterate(sd, fd, kern, 4.0, iters=3, check=False)
    assert r["rc"] == N.STPI_EINVAL and r["flags"] & 16 and r["iters"] == 0
    _, r = Sf.sfseg_iterate(sd, fd, kern, 1.0, iters=3)
    assert r["iters"] == 3 and not r["flags"]


@pytest.mark.parametrize("shape,kp,fscale,foff", [
    ((4, 31, 63), (4.0, 1.5, 8, 3), 1.0, 0.0), ((4, 32, 64), (3.0, 1.5, 7, 3), 1.0, 0.0),
    ((7, 33, 65), (4.0, 1.5, 5, 3), 1e-3, 0.0), ((3, 48, 66), (5.0, 2.0, 16, 5), 1.0, 0.0),
    ((13, 65, 67), (5.0, 2.0, 15, 5), 0.5, 3.0), ((12, 16, 130), (4.0, 2.0, 9, 4), 1e3, 0.0),
    ((2, 5, 3), (5.0, 2.0, 15, 5), 1.0, 0.0), ((9, 40, 72), (4.0, 1.5, 8, 3), 0.0, 0.0)])
def test_sfseg_matrix_core_step_and_chain(S, shape, kp, fscale, foff):
    """The matrix-core form around its tile edges, with f scaled and offset (its
    staging powers of two follow max |f|): one step per frame and eight
    iterations (uniform and given start, fixed count and tolerance chain) against
    the oracle. The update cancels terms of size max f^2 / (max f - min f)^2 above
    its result, so the float tolerance 1e-5 grows with that ratio."""
    P, Sf = S
    kern = P.Kernel(*kp)
    s, f = _fields(shape, 3)
    f = f * fscale + foff
    span = max(float(f.max() - f.min()), 1e-30)
    alpha = 0.9 / max(span * span, 1e-12)
    s, f = s.astype(np.float32), f.astype(np.float32)
    x = np.random.default_rng(9).uniform(-0.2, 1.0, shape).astype(np.float32)
    cond = max(1.0, alpha * float(np.max(f)) ** 2)
    sd, fd, xd = (torch.from_numpy(v).to(DEV) for v in (s, f, x))
    z, _ = Sf.sfseg_step(sd, fd, xd, kern, alpha, x_scale=0.3)
    torch.cuda.synchronize()
    ref = oracle.sfseg_apply(s.astype(np.float64), f.astype(np.float64), x.astype(np.float64) * 0.3, alpha, okf(kern))
    zz = z.double().cpu().numpy()
    for t in range(shape[0]):
        assert rel_l2(zz[t], ref[t]) <= 1e-5 * cond, (t, rel_l2(zz[t], ref[t]))
    x0 = np.abs(x) + np.float32(0.01)
    for start in (None, x0):
        kw = {} if start is None else dict(x0=torch.from_numpy(start).to(DEV))
        xg, r = Sf.sfseg_iterate(sd, fd, kern, alpha, iters=8, **kw)
        xg = xg.clone()
        xt, rt = Sf.sfseg_iterate(sd, fd, kern, alpha, tol=1e-300, max_iters=8, **kw)
        torch.cuda.synchronize()
        xr, info = oracle.sfseg_iterate(s, f, alpha, okf(kern), iters=8, x0=start)
        err = rel_l2(xg.double().cpu().numpy(), xr)
        print(shape, kp, fscale, foff, "chain", err)
        assert r["iters"] == 8 and err <= 1e-5 * cond
        assert abs(r["lambda_"] - info.lambdas[-1]) <= 1e-5 * cond * info.lambdas[-1]
        # the fixed-count chain skips the inner products it does not report
        assert torch.equal(xg, xt) and r["residual"] == rt["residual"] and r["r1"] == rt["r1"]


def test_sfseg_range_check_on_small_and_odd_volumes(S):
    """The range check's partial minima and maxima: volumes smaller than its
    grid, sizes that leave a tail after its 16-byte chunks, one bad voxel."""
    P, Sf = S
    kern = P.Kernel(1.0, 1.0, 1, 1)
    for shape in ((1, 1, 3), (3, 7, 11), (5, 64, 67)):
        n = int(np.prod(shape))
        s = torch.full(shape, 0.5, device=DEV)
        f = torch.linspace(0, 1, n, device=DEV).reshape(shape).contiguous()
        _, r = Sf.sfseg_iterate(s, f, kern, 1.0, iters=2)
        assert r["status"] == 0 and r["iters"] == 2
        for which, bad in (("s", -1e-3), ("s", float("nan")), ("f", 2.5), ("f", float("nan"))):
            for at in (0, n // 2, n - 1):
                v = dict(s=s.clone(), f=f.clone())
                v[which].view(-1)[at] = bad
                _, r = Sf.sfseg_iterate(v["s"], v["f"], kern, 1.0, iters=2, check=False)
                assert r["rc"] == 1 and r["flags"] & 16, (shape, which, bad, at)


def _one_iteration_at(P, Sf, s, f, x0, kern, alpha, idx):
    """(lambda x_1)_i of one iteration from x0 and its FP64 value, at the flat indices idx."""
    sd, fd, xd = (torch.from_numpy(v).to(DEV) for v in (s, f, x0))
    x, r = Sf.sfseg_iterate(sd, fd, kern, alpha, iters=1, x0=xd)
    torch.cuda.synchronize()
    got = x.double().cpu().numpy().reshape(-1)[idx] * r["lambda_"]
    x64 = x0.astype(np.float64)
    ref = oracle.sfseg_apply_at(s, f, x64 / np.linalg.norm(x64), alpha, okf(kern), idx)
    return got, ref


@pytest.mark.parametrize("shape,kp", [
    ((6, 64, 200), (5.0, 2.0, 15, 5)), ((5, 33, 140), (4.0, 2.0, 9, 4)), ((5, 60, 200), (4.0, 1.5, 8, 3)),
    ((5, 60, 200), (2.0, 1.0, 4, 2)),
    # either side of the volume from which r = (8, 3) takes its other form, and a smaller radius beyond it
    ((11, 464, 470), (4.0, 1.5, 8, 3)), ((12, 470, 470), (4.0, 1.5, 8, 3)), ((12, 470, 470), (4.0, 1.5, 6, 3)),
    # more workgroups than finalise their steps in the next launch
    ((2, 650, 1720), (2.0, 1.0, 4, 2)), ((2, 1040, 2060), (5.0, 2.0, 15, 5))])
def test_sfseg_keeps_float_precision_far_below_the_maximum(S, shape, kp):
    """s is 1 in the left columns and 1e-7, then 1e-14 further right: every voxel
    of an iteration keeps float's relative precision, also where a whole
    neighbourhood lies far below the volume's largest value. All terms of a
    voxel's sums are positive and the update cancels them by less than 5; the
    three passes round fewer than 80 times: 80 x 2^-24 x 5 per voxel."""
    P, Sf = S
    kern = P.Kernel(*kp)
    T, H, W = shape
    rng = np.random.default_rng(W)
    s = rng.uniform(0.5, 1.0, shape)
    s[:, :, 60:] *= 1e-7
    s[:, :, 110:] *= 1e-7
    s, f = s.astype(np.float32), rng.uniform(0.0, 0.9, shape).astype(np.float32)
    x0 = rng.uniform(0.5, 1.0, shape).astype(np.float32)
    cols = np.array([0, 20, 59, 60, 62, 76, 90, 109, 112, 126, W - 1])
    rows = rng.integers(0, H, 4)
    idx = np.array([(t * H + y) * W + c for t in (0, T - 1) for y in rows for c in cols])
    got, ref = _one_iteration_at(P, Sf, s, f, x0, kern, 1.0, idx)
    err = np.abs(got - ref) / np.abs(ref)
    print(shape, kp, "largest relative error", err.max(), "of values from", np.abs(ref).min(), "to", np.abs(ref).max())
    assert err.max() <= 80 * 2.0 ** -24 * 5


@pytest.mark.parametrize("kp", [(2.0, 1.0, 4, 2), (4.0, 1.5, 8, 3), (5.0, 2.0, 16, 5)])
@pytest.mark.parametrize("which,bad", [("x", float("nan")), ("x", float("inf")), ("s", float("nan")), ("f", float("inf"))])
def test_sfseg_step_keeps_non_finite_values_in_their_window(S, kp, which, bad):
    """A value that is not finite reaches the outputs whose window holds it and no others."""
    P, Sf = S
    kern = P.Kernel(*kp)
    shape, at = (13, 70, 150), (6, 33, 70)
    rng = np.random.default_rng(2)
    v = {k: torch.from_numpy(rng.uniform(0.1, 1.0, shape).astype(np.float32)).to(DEV) for k in "sfx"}
    clean, _ = Sf.sfseg_step(v["s"], v["f"], v["x"], kern, 1.0)
    clean = clean.clone()
    v[which][at] = bad
    z, _ = Sf.sfseg_step(v["s"], v["f"], v["x"], kern, 1.0)
    torch.cuda.synchronize()
    box = torch.zeros(shape, dtype=torch.bool, device=DEV)
    r_s, r_t = kp[2], kp[3]
    box[at[0] - r_t:at[0] + r_t + 1, at[1] - r_s:at[1] + r_s + 1, at[2] - r_s:at[2] + r_s + 1] = True
    assert torch.equal(z[~box], clean[~box])
    assert not torch.isfinite(z[box]).any()


def test_sfseg_infinite_feature_is_a_non_finite_iteration(S):
    """f infinite everywhere has no range to check: the iteration itself stops on its norm."""
    from paper_2212_08058_amd import _native as N
    P, Sf = S
    s = torch.full((4, 20, 30), 0.5, device=DEV)
    _, r = Sf.sfseg_iterate(s, torch.full_like(s, float("inf")), P.Kernel(5.0, 2.0, 15, 5), 1.0, iters=2, check=False)
    assert r["rc"] == 4 and r["flags"] & 2 and not r["flags"] & 16


@pytest.mark.parametrize("shape,kp", [((9, 40, 131), (4.0, 1.5, 8, 3)), ((9, 40, 131), (5.0, 2.0, 15, 5)),
                                      ((12, 470, 470), (4.0, 1.5, 8, 3)), ((7, 40, 131), (2.0, 1.0, 4, 2))])
def test_sfseg_finalisation_by_the_next_launch_is_bitwise_equal(S, monkeypatch, shape, kp):
    """The state formed by the next launch and the one formed by a launch of its
    own are the same, in the vector and the matrix-core form."""
    P, Sf = S
    kern = P.Kernel(*kp)
    rng = np.random.default_rng(5)
    s, f = (torch.from_numpy(rng.uniform(0.1, 1.0, shape).astype(np.float32)).to(DEV) for _ in range(2))
    out = []
    for flag in ("0", "1"):
        monkeypatch.setenv("STPI_NO_FUSE", flag)
        for kw in (dict(iters=5), dict(tol=1e-300, max_iters=19)):
            x, r = Sf.sfseg_iterate(s, f, kern, 1.0, **kw)
            torch.cuda.synchronize()
            out.append((x.clone(), {k: r[k] for k in ("iters", "residual", "lambda_", "rayleigh", "r1", "r2", "flags")}))
    for a, b in zip(out[:2], out[2:]):
        assert torch.equal(a[0], b[0]) and a[1] == b[1]

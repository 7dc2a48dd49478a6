"""lcsm_run_chain (stretches of chained steps in one launch) on the GPU
(needs an MI355X).

Where the shape allows (full state, at most 30 layers, at most 8192 columns
per layer) the chained steps of a stretch inside an aligned block of 32
positions whose gray tiles are direct tiles of U <= 16 run in one launch
that keeps the block's rows of every column in registers; the results must
equal the loop of single lcsm_step_chain calls bit for bit: one and several
layers (odd counts, and 30: sixteen waves), ragged shapes, lengths that are
not powers of two, the column-major mirror's tiles and stretches cut before
their block ends (direct tiles only up to U = 4, so the accumulators held in
registers go back to the state), every tile direct (the direct tiles of
U = 32 end a stretch), runs split into several calls at positions inside
blocks, and the shapes that take one position at a time (half-state
storage, more than 30 layers, more than 8192 columns).  Two shapes are also
checked against the fp64 oracle's closed loop."""
import numpy as np
import pytest
import torch

import datagen
from oracle import feedback
from oracle.relaxed import filters_to_columns, relaxed_online

from gpu_harness import TOL, dev, lcsm_mod, rel_err, say

pytestmark = pytest.mark.gpu

CASES = [
    ((1, 1, 16, 1024), None),
    ((3, 2, 33, 300), None),
    ((2, 3, 40, 2048), None),
    ((2, 4, 48, 2048), {"direct_max_u": 4, "col_fft_min_n": 16}),   # mirrored tiles from U = 8
    ((2, 2, 20, 700), {"direct_max_u": 1 << 20}),                   # every tile direct
    ((30, 1, 40, 300), None),                                       # sixteen waves
    ((18, 1, 64, 4096), None),
    ((2, 2, 24, 1200), {"half_state": 1}),                          # one position at a time
    ((34, 1, 8, 300), None),                                        # more layers than one launch takes
    ((1, 2, 4100, 200), None),                                      # more columns than one launch takes
    ((2, 1, 8, 1), None),                                           # one position, no tile
    ((1, 3, 8, 33), None),                                          # a last block of one position
]


def _ctx(w, opts):
    lcsm = lcsm_mod()
    h = datagen.filters_torch(w, dev())
    return lcsm.Lcsm(h, w.B, options=opts)


@pytest.mark.parametrize("shape,opts", CASES)
def test_run_chain_equals_single_steps(shape, opts):
    M, B, D, L = shape
    say(f"[run_chain] M={M} B={B} D={D} L={L} opts={opts}")
    w = datagen.Workload("chainrun", M, B, D, L, decay=L / 4, seed=M + 3 * B + D)
    x = datagen.x_torch(w, dev())
    ctx = _ctx(w, opts)
    z_ref = torch.empty_like(x)
    with torch.cuda.stream(ctx.stream):
        for t in range(L):
            ctx.step_chain(x[t], z_ref[t])
    torch.cuda.synchronize()
    ctx.reset()
    z = torch.full_like(x, float("nan"))
    ctx.run_chain(x, z)
    torch.cuda.synchronize()
    assert ctx.position == L
    assert torch.equal(z, z_ref)
    # in pieces that cut stretches in their middle
    ctx.reset()
    z2 = torch.full_like(x, float("nan"))
    cuts = [0, 5, 37, 38, 600, L]
    cuts = sorted({min(c, L) for c in cuts})
    for a, b in zip(cuts[:-1], cuts[1:]):
        ctx.run_chain(x[a:b], z2[a:b])
    torch.cuda.synchronize()
    assert torch.equal(z2, z_ref)
    ctx.close()


@pytest.mark.parametrize("M,BD", [(M, BD) for M in (1, 2, 3, 7, 8, 9, 16, 17, 22, 23, 30)
                                  for BD in (50, 4100)])
def test_run_chain_forms(M, BD):
    """Every form of the block launch at the edges of its layer counts (a lane
    per column up to 2 layers, then two halves of whole waves) and at 16 and 32
    columns per workgroup (above 4096 columns), last workgroup ragged: bit for
    bit the single steps, a run cut inside a block included."""
    say(f"[run_chain forms] M={M} BD={BD}")
    L, D = 100, BD // 2
    w = datagen.Workload("chainforms", M, 2, D, L, decay=L / 4, seed=M + BD)
    x = datagen.x_torch(w, dev())
    ctx = _ctx(w, None)
    z_ref, z = torch.empty_like(x), torch.full_like(x, float("nan"))
    with torch.cuda.stream(ctx.stream):
        for t in range(L):
            ctx.step_chain(x[t], z_ref[t])
        ctx.reset()
        ctx.run_chain(x[:45], z[:45])
        ctx.run_chain(x[45:], z[45:])
    torch.cuda.synchronize()
    assert torch.equal(z, z_ref)
    ctx.close()


@pytest.mark.parametrize("name", ["m1b1d16l1k", "layers4"])
def test_run_chain_matches_the_oracle_closed_loop(name):
    """The 1024-position workload, and 4 layers over 300 positions with
    fast-decaying filters: lengths over which an fp32 closed loop still
    follows the fp64 one (further on the chaotic loop amplifies rounding)."""
    w = (datagen.WORKLOADS[name] if name in datagen.WORKLOADS
         else datagen.Workload("chainrunref", 4, 2, 24, 300, decay=200.0, seed=25))
    M, B, D, L = w.M, w.B, w.D, w.L
    say(f"[run_chain vs oracle] M={M} B={B} D={D} L={L}")
    h = datagen.filters_np(w)
    x = datagen.x_np(w)
    ctx = lcsm_mod().Lcsm(torch.from_numpy(h).to(dev()), w.B)
    xd = torch.from_numpy(x).to(dev())
    z = torch.empty_like(xd)
    ctx.run_chain(xd, z)
    torch.cuda.synchronize()
    ctx.close()
    zr, _ = relaxed_online(filters_to_columns(h, w.B), feedback.tanh_chain(x.reshape(L, M, -1), M))
    err = rel_err(z.cpu().numpy().reshape(L, M, -1), zr)
    say(f"  rel err {err:.3e}")
    assert err <= TOL


@pytest.mark.parametrize("M,run", [(2, False), (2, True), (3, True), (9, False), (9, True)])
def test_chain_input_follows_the_emitted_z(M, run):
    """y^m = x^m + 0.5 tanh(z^{m-1}) of the z handed out, to the documented
    3.3e-7 for |x| <= 3, where z = h_0 y + acc cancels: layer 0 has taps (K, -K)
    and inputs by which z^0_1 = K (y^0_1 - y^0_0) stays small beside its terms,
    up to taps whose scaled sums would overflow; the other layers have the tap
    1 alone, so z^m is y^m.  One position a launch, a lane per column (M = 2)
    and the chain of a workgroup (M = 3, 9)."""
    say(f"[chain cancelling] M={M} run={run}")
    K = np.array([1.0, 10.0, 30.0, 100.0, 1e4, 2e38]).repeat(128)
    B, D, L = 4, K.size, 4
    rng = np.random.default_rng(5)
    h = np.zeros((M, D, L), np.float32)
    h[0, :, 0], h[0, :, 1] = K, -K
    h[1:, :, 0] = 1.0
    x = rng.uniform(-1, 1, (2, M, B, D)).astype(np.float32)
    x[0, 0] = rng.uniform(0.3, 0.9, (B, D))
    # x^0_1 such that y^0_1 = y^0_0 + delta, |K delta| <= 1
    z = K * x[0, 0].astype(np.float64)
    for m in range(1, M):
        z = x[0, m] + 0.5 * np.tanh(z)
    x[1, 0] = x[0, 0] + rng.uniform(-1, 1, (B, D)) / K - 0.5 * np.tanh(z)
    assert np.abs(x).max() <= 3
    ctx = lcsm_mod().Lcsm(torch.from_numpy(h).to(dev()), B)
    xd = torch.from_numpy(x).to(dev())
    zd = torch.full_like(xd, float("nan"))
    if run:
        ctx.run_chain(xd, zd)
    else:
        for t in range(2):
            ctx.step_chain(xd[t], zd[t])
    torch.cuda.synchronize()
    ctx.close()
    zg = zd.cpu().numpy().astype(np.float64)
    err = np.abs(zg[:, 1:] - (x[:, 1:] + 0.5 * np.tanh(zg[:, :-1])))
    for k in range(6):
        say(f"  K={K[128 * k]:g}: max |z^0_1| {np.abs(zg[1, 0, :, 128 * k:128 * k + 128]).max():.3g}, "
            f"error of y {err[..., 128 * k:128 * k + 128].max():.3e}")
    assert err.max() < 3.3e-7


@pytest.mark.parametrize("M", [1, 2, 3, 9])
@pytest.mark.parametrize("ahead", [1, 2, 5, 31, 32, -1, 0])
def test_run_chain_reads_back_its_outputs(M, ahead):
    """x_{k+ahead} is z_k (one buffer, z `ahead` slabs behind x): the block
    launch loads x ahead, so it may not take such positions.  The loop of single
    steps is the reference; ahead <= 0 overwrites inputs already read."""
    say(f"[run_chain reads back] M={M} ahead={ahead}")
    B, D, L = 2, 40, 100
    w = datagen.Workload("chainback", M, B, D, L, decay=8.0, seed=M + ahead)
    ctx = lcsm_mod().Lcsm(datagen.filters_torch(w, dev()) * 0.1, B)
    slab, lead = M * B * D, max(0, -ahead)
    x0 = torch.rand((L + 32, M, B, D), device=dev()) - 0.5
    want, got = x0.clone(), x0.clone()
    xs, zs = 4 * slab * lead, 4 * slab * (lead + ahead)
    lib = lcsm_mod().raw()
    for t in range(L):
        p = want.data_ptr() + 4 * slab * t
        assert lib.lcsm_step_chain(ctx._ctx, p + xs, p + zs) == 0
    ctx.reset()
    assert lib.lcsm_run_chain(ctx._ctx, L, got.data_ptr() + xs, slab, got.data_ptr() + zs, slab) == 0
    torch.cuda.synchronize()
    assert torch.isfinite(want).all()
    assert torch.equal(got, want)
    ctx.close()


@pytest.mark.parametrize("M,ring", [(1, 3), (2, 31), (9, 1), (9, 3), (9, 40)])
def test_recorded_chain_on_one_ring(M, ring):
    """A recorded run whose x and z are one ring: step k reads what step k - ring
    wrote."""
    say(f"[run_chain ring] M={M} ring={ring}")
    B, D, L = 2, 40, 100
    w = datagen.Workload("chainring", M, B, D, L, decay=8.0, seed=M + ring)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        ctx = lcsm_mod().Lcsm(datagen.filters_torch(w, dev()) * 0.1, B)
        x0 = torch.rand((ring, M, B, D), device=dev()) - 0.5
        want, got = x0.clone(), x0.clone()
        for t in range(L):
            ctx.step_chain(want[t % ring], want[t % ring])
        g = ctx.capture(got, got, n=L, chain=True)
        g.launch()
    torch.cuda.synchronize()
    assert torch.isfinite(want).all()
    assert torch.equal(got, want)
    ctx.close()


def test_run_chain_errors():
    lcsm = lcsm_mod()
    w = datagen.Workload("chainrunerr", 1, 1, 8, 40, decay=10.0, seed=2)
    x = datagen.x_torch(w, dev())
    ctx = _ctx(w, None)
    z = torch.empty_like(x)
    ctx.run_chain(x, z)
    with pytest.raises(lcsm.LcsmError) as e:
        ctx.run_chain(x[:1], z[:1])
    assert e.value.code == lcsm.LCSM_EDONE
    lib = lcsm.raw()
    assert lib.lcsm_run_chain(None, 1, x.data_ptr(), 8, z.data_ptr(), 8) == lcsm.LCSM_EINVAL
    ctx.reset()
    assert lib.lcsm_run_chain(ctx._ctx, -1, x.data_ptr(), 8, z.data_ptr(), 8) == lcsm.LCSM_EINVAL
    assert lib.lcsm_run_chain(ctx._ctx, 0, x.data_ptr(), 8, z.data_ptr(), 8) == lcsm.LCSM_OK
    ctx.close()

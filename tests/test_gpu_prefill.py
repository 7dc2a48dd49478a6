"""GPU parity of the prompt prefill (lcsm_prefill; needs an MI355X).

With all P prompt inputs known, the prompt's outputs come from one 2P-point
transform (the filter delayed by P rows), and the context is left exactly as
P online steps would leave it; the generation then continues step by step.
Bars: the whole run (prompt plus generation) against the fp64 static-FFT
oracle on the same teacher-forced inputs, max|z_gpu - z_ref| <= 1e-4 *
max|z_ref|; on small-integer data the rounded outputs equal the exact int64
convolution.
"""
import numpy as np
import pytest
import torch

import datagen
from oracle import conv
from oracle.relaxed import filters_to_columns

from gpu_harness import TOL, dev, lcsm_mod, make_ctx, rel_err, say

pytestmark = pytest.mark.gpu

OPTIONS = {
    "default": None,
    # every tile above U = 1 is an FFT tile, one LDS pass up to 2U = 4096
    "fft_from_2": {"direct_max_u": 1, "lds_fft_max_n": 4096, "col_fft_min_n": 1 << 20},
    # every tile with 2U > 16 (and the prompt's transform) in three passes
    "multipass_from_16": {"direct_max_u": 1, "lds_fft_max_n": 16, "col_fft_min_n": 1 << 20},
    # every FFT tile (and the prompt's transform) on transposed column chunks
    "col_from_4": {"direct_max_u": 1, "col_fft_min_n": 4},
    "colT_from_4": {"direct_max_u": 1, "col_fft_min_n": 4, "col_tile_form": 1},
}


def _prefill_then_run(ctx, y, P):
    z = torch.full_like(y, float("nan"))
    ctx.prefill(y[:P], z[:P])
    assert ctx.position == P
    if y.shape[0] > P:
        ctx.run(y[P:], z[P:])
    torch.cuda.synchronize()
    return z.cpu().numpy()


@pytest.mark.parametrize("opt", ["default", "fft_from_2", "multipass_from_16", "col_from_4",
                                 "colT_from_4"])
@pytest.mark.parametrize("case", [(2, 3, 40, 1024, 256), (3, 2, 33, 2048, 64), (1, 1, 5, 300, 128),
                                  (2, 2, 24, 4096, 2048), (1, 2, 8, 32768, 16384)])
def test_prefill_then_generate_matches_oracle(opt, case):
    """The last case's prompt tile is 2U = 32768: with column tiles it runs as
    the two 16384-point halves, with the filter spectrum delayed by P."""
    M, B, D, L, P = case
    w = datagen.Workload("prefill", M, B, D, L, decay=L / 4, seed=31 + P)
    say(f"[prefill] M={M} B={B} D={D} L={L} P={P} options={opt}")
    ctx, _ = make_ctx(w, options=OPTIONS[opt])
    y = datagen.y_torch(w, dev())
    z = _prefill_then_run(ctx, y, P)
    h = filters_to_columns(datagen.filters_np(w), w.B)
    zr = conv.causal_conv_fft(y.cpu().numpy().reshape(L, -1).astype(np.float64), h.reshape(h.shape[0], -1))
    err_prompt = rel_err(z[:P].reshape(P, -1), zr[:P])
    err = rel_err(z.reshape(L, -1), zr)
    say(f"  rel err prompt {err_prompt:.3e}, whole run {err:.3e}")
    assert err <= TOL


def test_prefill_bench_workload_half_prompt():
    """m1b8d768l8k with a 4096-position prompt (the 2U = 8192 transform for
    the prompt's outputs), then 4096 online steps."""
    w = datagen.WORKLOADS["m1b8d768l8k"]
    P = w.L // 2
    say(f"[prefill] {w.name} P={P}")
    ctx, _ = make_ctx(w)
    y = datagen.y_torch(w, dev())
    z = _prefill_then_run(ctx, y, P)
    h = filters_to_columns(datagen.filters_np(w), w.B)
    zr = conv.causal_conv_fft(y.cpu().numpy().reshape(w.L, -1).astype(np.float64), h.reshape(h.shape[0], -1))
    err = rel_err(z.reshape(w.L, -1), zr)
    say(f"  rel err {err:.3e}")
    assert err <= TOL


@pytest.mark.parametrize("opt", ["default", "multipass_from_16", "col_from_4"])
def test_prefill_integer_data_rounds_to_exact(opt):
    M, B, D, L, P = 2, 2, 16, 2048, 512
    w = datagen.Workload("int", M, B, D, L, decay=1.0, seed=7)
    h = datagen.int_filters_np(w, 3)
    y = datagen.int_y_np(w, 3)
    say(f"[prefill int] M={M} B={B} D={D} L={L} P={P} options={opt}")
    ctx, _ = make_ctx(w, torch.from_numpy(h).to(dev()), OPTIONS[opt])
    z = _prefill_then_run(ctx, torch.from_numpy(y).to(dev()), P)
    ex = np.zeros((L, M, B, D), dtype=np.int64)
    hi, yi = h.astype(np.int64), y.astype(np.int64)
    for k in range(L):
        ex[k:] += yi[: L - k] * hi[None, :, None, :, k]
    assert np.abs(z.astype(np.float64) - ex).max() < 0.25
    assert np.array_equal(np.rint(z).astype(np.int64), ex)


def test_prefill_continues_like_stepwise_run_and_reset_repeats():
    """Prefill + steps against all steps on the same inputs (the two orders of
    summation agree to fp32 rounding), and a reset context prefills again to
    the same bits."""
    w = datagen.Workload("prefill2", 2, 2, 48, 2048, decay=512.0, seed=5)
    P = 512
    ctx, _ = make_ctx(w)
    y = datagen.y_torch(w, dev())
    za = _prefill_then_run(ctx, y, P)
    ctx.reset()
    zb = torch.empty_like(y)
    ctx.run(y, zb)
    torch.cuda.synchronize()
    zb = zb.cpu().numpy()
    assert rel_err(za, zb.astype(np.float64)) <= 1e-5
    ctx.reset()
    zc = _prefill_then_run(ctx, y, P)
    assert np.array_equal(za, zc)


def test_prefill_errors():
    lcsm = lcsm_mod()
    w = datagen.Workload("prefill3", 1, 1, 8, 256, decay=64.0, seed=3)
    ctx, _ = make_ctx(w)
    y = datagen.y_torch(w, dev())
    z = torch.empty_like(y)
    for P in (0, 3, 96, 256):  # not a power of two, or 2P > L
        with pytest.raises(lcsm.LcsmError) as ex:
            ctx.prefill(y[:max(P, 1)] if P else y[:1], z, P=P)
        assert ex.value.code == lcsm.LCSM_EINVAL
    ctx.step(y[0], z[0])
    with pytest.raises(lcsm.LcsmError) as ex:
        ctx.prefill(y[:64], z[:64])
    assert ex.value.code == lcsm.LCSM_ESTATE
    ctx.reset()
    ctx.prefill(y[:128], z[:128])
    assert ctx.position == 128


@pytest.mark.parametrize("case", [
    # (M, B, D, L, P, options, extra floats per position slab, first slab moved by floats)
    (3, 2, 64, 512, 64, {}, 0, 0),            # 16-byte copies, pairs of batch rows
    (3, 2, 64, 512, 64, {}, 4, 0),
    (3, 2, 64, 512, 64, {}, 2, 0),            # slabs that are not 16-byte apart
    (3, 2, 64, 512, 64, {}, 0, 1),            # nor aligned
    (2, 3, 37, 500, 32, {}, 1, 0),            # neighbouring columns, the last one alone
    (2, 1, 128, 300, 2, {}, 0, 0),            # the smallest mirrored prompt
    (5, 1, 33, 4100, 2048, {"scratch_mib": 2}, 0, 0),  # two layers' spectra at a time
    (1, 1, 1, 1024, 256, {}, 0, 0),           # one column: the spectra do not fit the scratch
    (1, 2, 6, 32768, 16384, {}, 0, 0),        # the prompt's transform as two halves
    (1, 2, 4, 70000, 1024, {}, 0, 0),         # larger tiles read the prompt from the state
])
def test_prefill_on_the_mirror(case):
    """The prompt of a mirrored tile size (mirror forced from 2U = 4): inputs
    straight into the mirror, delayed spectra by chunks of layers, outputs
    straight out of it; then the generation goes on."""
    M, B, D, L, P, opts, pad, move = case
    say(f"[prefill mirror] {case}")
    w = datagen.Workload("prefill_cm", M, B, D, L, decay=max(L / 8, 8.0), seed=7 + P)
    ctx, _ = make_ctx(w, options={"direct_max_u": 1, "col_fft_min_n": 4, **opts})
    n = min(L, 2 * P + 70) if L < 70000 else L
    y = datagen.y_torch(w, dev())[:n].contiguous()
    slab = M * B * D
    ys = torch.zeros(P * (slab + pad) + move, device=dev())
    zs = torch.full_like(ys, float("nan"))
    rows = ys[move:].view(P, slab + pad)
    rows[:, :slab] = y[:P].reshape(P, slab)
    z = torch.full_like(y, float("nan"))
    r = lcsm_mod().raw().lcsm_prefill(ctx._ctx, P, ys.data_ptr() + 4 * move, slab + pad,
                                      zs.data_ptr() + 4 * move, slab + pad)
    assert r == 0
    ctx.run(y[P:], z[P:])
    torch.cuda.synchronize()
    out = zs[move:].view(P, slab + pad)
    assert torch.isnan(out[:, slab:]).all()  # nothing written between the slabs
    z[:P] = out[:, :slab].reshape(P, M, B, D)
    h = filters_to_columns(datagen.filters_np(w), B)[:n]
    zr = conv.causal_conv_fft(y.cpu().numpy().reshape(n, -1).astype(np.float64), h.reshape(n, -1))
    err = rel_err(z.cpu().numpy().reshape(n, -1), zr)
    say(f"  rel err {err:.3e}")
    # sums over at most 16 levels of tiles, each within about 10 roundings of its 2U-point transforms
    assert err <= 16 * 10 * 2.0 ** -24
    ctx.close()


@pytest.mark.parametrize("case", [
    # (M, B, D, L, P, scratch_mib of the second context)
    (3, 2, 5, 512, 64, 0),
    (2, 3, 37, 500, 32, 0),
    (4, 2, 1, 300, 128, 0),           # one channel a layer
    (5, 1, 33, 4100, 2048, 2),        # two layers' spectra at a time
    (2, 2, 3, 32768, 16384, 0),       # the transform as two halves
])
def test_mirrored_prompt_keeps_layers_apart(case):
    """Odd D: the last channel of a layer shares its delayed spectrum's
    transform with no channel of the next layer.  Whatever layer 0's taps are
    (10^4 times as large, one of them not finite), the other layers' prompt
    outputs and the steps behind them keep their bits, and so does everything
    where the layers are taken in other chunks."""
    M, B, D, L, P, mib = case
    say(f"[prefill layers apart] {case}")
    w = datagen.Workload("prefill_la", M, B, D, L, decay=max(L / 8, 8.0), seed=11 + P)
    n = P + 70
    y = datagen.y_torch(w, dev())[:n].contiguous()
    h = datagen.filters_torch(w, dev())

    def run(filters, **opts):
        ctx, _ = make_ctx(w, filters, {"direct_max_u": 1, "col_fft_min_n": 4, **opts})
        z = torch.full_like(y, float("nan"))
        ctx.prefill(y[:P], z[:P])
        ctx.run(y[P:], z[P:])
        torch.cuda.synchronize()
        ctx.close()
        return z

    z = run(h)
    assert torch.isfinite(z).all()
    large, bad = h.clone(), h.clone()
    large[0] *= 1e4
    bad[0, D - 1, 3] = float("nan")
    assert torch.equal(run(large)[:, 1:], z[:, 1:])
    zb = run(bad)
    assert torch.equal(zb[:, 1:], z[:, 1:])
    assert torch.isnan(zb[3:P, 0, :, D - 1]).all()
    if mib:
        assert torch.equal(run(h, scratch_mib=mib), z)


@pytest.mark.parametrize("P", [1024, 2048, 4096, 8192, 16384])
def test_mirrored_prompt_is_as_exact_as_the_general_path(P):
    """The prompt's outputs against 64 bits: the mirror's delayed spectra add no
    more rounding than those of the general path (transposed chunks), whose
    transforms are the same otherwise.  The 2-norm runs over 10^6 outputs and
    more, so two such norms of like errors differ by well below 1 %."""
    M, B, D = 2, 2, max(16, (1 << 18) // P)
    say(f"[prefill precision] P={P}")
    w = datagen.Workload("prefill_pr", M, B, D, 2 * P, decay=P / 2, seed=17 + P)
    y = datagen.y_torch(w, dev())[:P].contiguous()
    h = filters_to_columns(datagen.filters_np(w), B)[:P]
    zr = conv.causal_conv_fft(y.cpu().numpy().reshape(P, -1).astype(np.float64), h.reshape(P, -1))
    err = {}
    for form in (0, 1):
        ctx, _ = make_ctx(w, options={"direct_max_u": 1, "col_fft_min_n": 4, "col_tile_form": form})
        z = torch.full_like(y, float("nan"))
        ctx.prefill(y, z)
        torch.cuda.synchronize()
        ctx.close()
        d = z.cpu().numpy().reshape(P, -1).astype(np.float64) - zr
        err[form] = float(np.linalg.norm(d) / np.linalg.norm(zr))
    say(f"  rel err mirror {err[0]:.4e}, general path {err[1]:.4e}")
    assert err[0] <= 1.02 * err[1]

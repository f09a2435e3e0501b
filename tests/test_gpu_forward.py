"""GPU parity of the forward path: HIP kernels vs the FP64 oracle, element by
element on the same seeded inputs (the oracle reads the dequantised stored
values), gate err_inf <= 1e-5 per component; plus the bit-exact loader."""

import numpy as np
import pytest
import torch

import oracle
from paper_2607_01338_amd import metrics as M
from paper_2607_01338_amd import rt
from paper_2607_01338_amd import workloads as W

from gpu_helpers import (TOL_FWD, dequantised, gpu_forward, line_dict, problem, say, to_device)

pytestmark = pytest.mark.gpu


def check_cube(cube, dt, line=None, pix=None, tol=TOL_FWD, label=""):
    line = line or dict(W.LINE_13CO_21)
    say(f"[fwd] {label or cube.name} shape={cube.shape} axis={cube.axis} dtype={dt} "
        f"C={cube.channels.n_chan}")
    dev = to_device(cube, dt)
    out = gpu_forward(cube, dev, line)
    deq = dequantised(dev)
    ref = oracle.forward(problem(cube, deq), line, pix=pix)
    errs = {}
    # A component far below the cube's own scale (e.g. a background behind
    # e^-600 of dust, below FP32 range) is gated in absolute terms at
    # TOL * 1e-6 * max|[T]|.
    floor = 1e-6 * float(np.max(np.abs(ref["T"])))
    for k in "TCDLB":
        g = out[k].double().cpu().numpy()
        if pix is not None:
            g = g[pix.start:pix.stop] if isinstance(pix, range) else g[pix]
        errs[k] = M.err_inf(g, ref[k], floor)
    say(f"      err_inf {errs}")
    for k, e in errs.items():
        assert e <= tol, (k, e)
    return out, ref


def test_small_config_fp64_full():
    check_cube(W.config_small(), "f64")


@pytest.mark.parametrize("dt", ["f32", "f64", "bf16", "f16"])
def test_ragged_along_y(dt):
    # 100 cells per sightline: one full 64-cell chunk plus a ragged tail;
    # 150 channels: windows straddle the 64-lane passes and the channel end.
    cube = W.make_cube((6, 100, 5), 1, W.Channels(150, -30.0, 0.4), seed=21, v_rms_kms=12.0)
    check_cube(cube, dt)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_ragged_along_x(dt):
    cube = W.make_cube((130, 3, 4), 0, W.Channels(96, -48.0, 1.0), seed=22, v_rms_kms=20.0)
    check_cube(cube, dt)


def test_long_sightlines_wide_band():
    # CMZ-like sightlines: 512 cells, 800 channels of 0.5 km/s over +-200 km/s.
    cube = W.make_cube((3, 512, 5), 1, W.CH_C2, seed=23, v_rms_kms=90.0)
    check_cube(cube, "f32")


def test_separate_dust_temperature_and_strong_dust():
    cube = W.make_cube((4, 5, 70), 2, W.Channels(64, -32.0, 1.0), seed=24, t_dust=True)
    check_cube(cube, "f32", line_dict(kappa_dust_cm2g=300.0))


def test_literal_upper_energy_mode():
    cube = W.make_cube((4, 5, 40), 2, W.Channels(48, -24.0, 1.0), seed=25)
    check_cube(cube, "f32", line_dict(energy_mode=1))


def test_dust_thick_chunks_rebase():
    # Dust optical depth ~0.2-20 per cell: the scaled state is rebased many
    # times inside a 64-cell chunk.
    cube = W.make_cube((3, 4, 90), 2, W.Channels(40, -20.0, 1.0), seed=26)
    out, ref = check_cube(cube, "f32", line_dict(kappa_dust_cm2g=3e4))
    assert np.min(ref["B"]) < 1e-3 * W.LINE_13CO_21["t_bg_k"]


@pytest.mark.parametrize("xscale", [1e-2, 1e-3, 1e-5])
def test_faint_lines_per_sightline(xscale):
    # Faint lines: the continuum sits far from the line source function, so
    # each in-window step changes the excess by a small part of its size. The
    # gate is taken per sightline, against that sightline's own maximum, for
    # the total and the line ([T] ~ 4 K, [L] ~ 0.2 K at 1e-3 of the abundance).
    cube = W.make_cube((4, 5, 384), 2, W.Channels(300, -75.0, 0.5), seed=211, v_rms_kms=25.0)
    say(f"[fwd] faint lines, abundance x {xscale}")
    dev = to_device(cube, "f32")
    dev["x_tracer"] = dev["x_tracer"] * xscale
    out = gpu_forward(cube, dev)
    ref = oracle.forward(problem(cube, dequantised(dev)), dict(W.LINE_13CO_21))
    for k in "TL":
        g = out[k].double().cpu().numpy()
        scale = np.maximum(np.abs(ref[k]).max(axis=1), 1e-3 * np.abs(ref[k]).max())
        per = np.abs(g - ref[k]).max(axis=1) / scale
        say(f"      [{k}] max {np.abs(ref[k]).max():.3g}, worst per-sightline err {per.max():.3g}")
        assert per.max() <= TOL_FWD, (k, per.max())


@pytest.mark.parametrize("integrator,transfer", [("smooth", "thick"), ("formal", "thin"),
                                                 ("formal", "selective"), ("smooth", "selective")])
def test_faint_lines_per_sightline_other_modes(integrator, transfer):
    # The same faint-line gate for the smooth integrator and the thin modes, at
    # 1e-3 of the abundance (at 1e-5, [L] ~ 2 mK, the smooth kernels' per-sightline
    # error reaches 5e-5 of that, about 0.1 microkelvin).
    cube = W.make_cube((4, 5, 384), 2, W.Channels(300, -75.0, 0.5), seed=211, v_rms_kms=25.0)
    say(f"[fwd] faint lines, {integrator} / {transfer}")
    dev = to_device(cube, "f32")
    dev["x_tracer"] = dev["x_tracer"] * 1e-3
    line = line_dict(integrator=integrator, transfer=transfer)
    out = gpu_forward(cube, dev, line)
    ref = oracle.forward(problem(cube, dequantised(dev)), line)
    for k in "TL":
        g = out[k].double().cpu().numpy()
        scale = np.maximum(np.abs(ref[k]).max(axis=1), 1e-3 * np.abs(ref[k]).max())
        per = np.abs(g - ref[k]).max(axis=1) / scale
        say(f"      [{k}] worst per-sightline err {per.max():.3g}")
        assert per.max() <= TOL_FWD, (k, per.max())


def test_edge_cases_single_cell_single_channel():
    cube = W.make_cube((3, 4, 1), 2, W.Channels(1, -0.5, 1.0), seed=27, v_rms_kms=0.3)
    check_cube(cube, "f32")
    cube = W.make_cube((2, 1, 3), 1, W.Channels(7, -3.5, 1.0), seed=28, v_rms_kms=2.0)
    check_cube(cube, "f32")


def test_edge_cases_hot_empty_and_out_of_band():
    cube = W.make_cube((4, 4, 33), 2, W.Channels(64, -16.0, 0.5), seed=29, v_rms_kms=40.0)
    cube.t_kin[:, :, ::3] = 80.0            # above T_inf below
    cube.x_tracer[:, :, 1::5] = 0.0         # no tracer
    cube.v_los[0, :, :] = 500.0             # far outside the band
    check_cube(cube, "f32", line_dict(t_inf_k=60.0, t_bg_k=0.0))


def test_deterministic_bitwise():
    cube = W.make_cube((5, 6, 77), 2, W.Channels(130, -40.0, 0.6), seed=30)
    dev = to_device(cube, "f32")
    a = gpu_forward(cube, dev)
    b = gpu_forward(cube, dev)
    for k in "TCDLB":
        assert torch.equal(a[k], b[k]), k


def test_outputs_can_be_skipped():
    cube = W.make_cube((2, 3, 20), 2, W.Channels(32, -16.0, 1.0), seed=31)
    dev = to_device(cube, "f32")
    full = gpu_forward(cube, dev)
    part = gpu_forward(cube, dev, components="L")
    assert set(part) == {"L"}
    assert torch.equal(part["L"], full["L"])


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_layout_bit_exact(axis, dt):
    cube = W.make_cube((70, 67, 9), axis, W.Channels(8, -4, 1), seed=32, t_dust=True)
    say(f"[layout] axis={axis} dtype={dt}")
    dev = to_device(cube, dt)
    soa = rt.iris_rt_layout(dev["ln_nh2"], dev["t_kin"], dev["v_los"], dev["x_tracer"],
                            dev["t_dust"], axis=axis)
    torch.cuda.synchronize()
    for i, k in enumerate(("ln_nh2", "t_kin", "v_los", "x_tracer", "t_dust")):
        a = dev[k].cpu()
        ref = a.movedim(axis, 2).reshape(-1, a.shape[axis])
        assert torch.equal(soa[i].cpu().view(torch.int8), ref.contiguous().view(torch.int8)), k


# --- full-size CMZ cube, sampled against the oracle --------------------------

@pytest.fixture(scope="module")
def cmz_cube():
    say("[fwd] generating the 512x512x128 CMZ cube")
    return W.config_cmz()


@pytest.mark.parametrize("dt", ["f32", "bf16", "f16"])
def test_cmz_full_size_sampled(cmz_cube, dt):
    rng = np.random.default_rng(40)
    pix = np.sort(rng.choice(cmz_cube.n_pix, 48, replace=False))
    say(f"[fwd] CMZ 512x512x128 along y, 800 ch, dtype={dt}, 48 sampled sightlines")
    dev = to_device(cmz_cube, dt)
    out = gpu_forward(cmz_cube, dev)
    deq = dequantised(dev)
    del dev
    pr = problem(cmz_cube, deq)
    errs = {k: 0.0 for k in "TCDLB"}
    refs = {k: [] for k in "TCDLB"}
    for p in pix:
        ref = oracle.forward(pr, W.LINE_13CO_21, pix=range(int(p), int(p) + 1))
        for k in "TCDLB":
            refs[k].append(ref[k][0])
    for k in "TCDLB":
        g = out[k][torch.from_numpy(pix).cuda()].double().cpu().numpy()
        errs[k] = M.err_inf(g, np.array(refs[k]))
    say(f"      err_inf {errs}")
    for k, e in errs.items():
        assert e <= TOL_FWD, (k, e)
    # Sanity of the physics at scale: emission present, non-negative totals.
    T = out["T"]
    assert float(T.max()) > 5.0 and float(T.min()) >= 0.0


@pytest.mark.parametrize("axis", [0, 1])
def test_in_place_reads_match_transposed_copy(axis, monkeypatch):
    # Fields along x or y are read in place by default; the sightline-major
    # copy is the same values in another order, so every output must be
    # bit-identical between the two.
    shape = (70, 9, 33) if axis == 0 else (9, 70, 33)
    cube = W.make_cube(shape, axis, W.Channels(96, -24.0, 0.5), seed=77, v_rms_kms=6.0)
    dev = to_device(cube, "f32")
    say(f"[fwd] in place vs transposed copy, axis={axis}")
    a = gpu_forward(cube, dev)
    monkeypatch.setenv("IRIS_RT_FIELD_LAYOUT", "transpose")
    b = gpu_forward(cube, dev)
    for k in "TCDLB":
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("groups", [1, 2, 4])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_every_sightline_packing(groups, dt, monkeypatch):
    # 1, 2 or 4 sightlines per wavefront, forced: 7 x 5 = 35 sightlines (not a
    # multiple of the packing, so the last wavefront is partly empty), wide
    # enough windows for several passes at 16 lanes, thick dust to rebase.
    monkeypatch.setenv("IRIS_RT_SIGHTLINES_PER_WAVE", str(groups))
    cube = W.make_cube((7, 5, 150), 2, W.Channels(120, -30.0, 0.5), seed=90 + groups,
                       v_rms_kms=8.0)
    check_cube(cube, dt, line_dict(kappa_dust_cm2g=300.0), label=f"G={groups}")


def test_unaligned_outputs_match_aligned():
    # Rows of 96 channels written through 16-byte stores when every output is
    # 16-byte aligned; output views offset by one float take the per-channel
    # stores. Same arithmetic, so the cubes must be bit-identical.
    cube = W.make_cube((5, 6, 40), 2, W.Channels(96, -24.0, 0.5), seed=79, v_rms_kms=6.0)
    dev = to_device(cube, "f32")
    say("[fwd] 16-byte vs unaligned output stores")
    a = gpu_forward(cube, dev)
    n_pix, C = cube.n_pix, cube.channels.n_chan
    dev0 = dev["ln_nh2"].device
    flat = {k: torch.full((n_pix * C + 1,), -1.0, dtype=torch.float32, device=dev0) for k in "TCDLB"}
    out = {k: flat[k][1:].view(n_pix, C) for k in "TCDLB"}
    rt.iris_rt_forward(dev["ln_nh2"], dev["t_kin"], dev["v_los"], dev["x_tracer"], axis=cube.axis,
                       cell_cm=cube.cell_cm, channels=rt.Channels(C, cube.channels.v_lo_kms,
                                                                  cube.channels.dv_kms),
                       out=out)
    torch.cuda.synchronize()
    for k in "TCDLB":
        assert float(flat[k][0]) == -1.0, k  # nothing written before the view
        assert torch.equal(a[k], out[k]), k


@pytest.mark.parametrize("units", ["intensity", "tb"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_output_units(units, dt):
    # Specific intensity (every component scaled) and Planck brightness
    # temperature ([T], [C], [B]; [L], [D] stay Rayleigh-Jeans) against the
    # oracle in the same units; thick dust drives [B] towards zero.
    cube = W.make_cube((4, 5, 60), 2, W.Channels(96, -24.0, 0.5), seed=80, v_rms_kms=6.0)
    check_cube(cube, dt, line_dict(units=units, kappa_dust_cm2g=200.0), label=f"units={units}")


def test_intensity_units_scale_the_kelvin_cubes():
    # Same march, output scaled by one factor: every component of the
    # intensity cube is the kelvin cube times 2 k nu0^2 / c^2 (to FP32
    # rounding of the product).
    cube = W.make_cube((3, 4, 30), 2, W.Channels(64, -16.0, 0.5), seed=81, v_rms_kms=5.0)
    dev = to_device(cube, "f32")
    a = gpu_forward(cube, dev, line_dict())
    b = gpu_forward(cube, dev, line_dict(units="intensity"))
    s = 2 * 1.380649e-16 * W.LINE_13CO_21["nu0_hz"] ** 2 / 2.99792458e10 ** 2
    for k in "TCDLB":
        ref = a[k].double() * s
        err = float((b[k].double() - ref).abs().max() / ref.abs().max().clamp_min(1e-300))
        assert err < 1e-6, (k, err)


def _subsampled_problem(cube, deq, f):
    ch = cube.channels
    return oracle.Problem(deq["ln_nh2"], deq["t_kin"], deq["v_los"], deq["x_tracer"], cube.axis,
                          cube.cell_cm, ch.n_chan, ch.v_lo_kms, ch.dv_kms, deq.get("t_dust"),
                          simpson_f=f)


@pytest.mark.parametrize("f", [1, 2])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_velocity_subsampling(f, dt):
    # Fine grid of 2 f C + 1 velocities marched, channels reported as their
    # composite-Simpson averages; narrow lines (b ~ 1.4 dv) so that the
    # averaging matters; against the oracle on the same grid.
    cube = W.make_cube((4, 5, 50), 2, W.Channels(48, -24.0, 1.0), seed=84, v_rms_kms=6.0)
    dev = to_device(cube, dt)
    say(f"[fwd] subsampled f={f} dtype={dt}")
    ch = cube.channels
    out = rt.iris_rt_forward(dev["ln_nh2"], dev["t_kin"], dev["v_los"], dev["x_tracer"],
                             axis=cube.axis, cell_cm=cube.cell_cm,
                             channels=rt.Channels(ch.n_chan, ch.v_lo_kms, ch.dv_kms, f))
    torch.cuda.synchronize()
    ref = oracle.forward(_subsampled_problem(cube, dequantised(dev), f), dict(W.LINE_13CO_21))
    floor = 1e-6 * float(np.max(np.abs(ref["T"])))
    errs = {k: M.err_inf(out[k].double().cpu().numpy(), ref[k], floor) for k in "TCDLB"}
    say(f"      err_inf {errs}")
    for k, e in errs.items():
        assert e <= TOL_FWD, (k, e)
    # The averaging changes the cube: centre sampling differs at this width.
    centre = oracle.forward(problem(cube, dequantised(dev)), dict(W.LINE_13CO_21))
    assert np.max(np.abs(centre["L"] - ref["L"])) > 1e-3 * np.max(np.abs(ref["L"]))


@pytest.mark.parametrize("dt", ["f32", "bf16", "f64"])
def test_check_fields_counts_unusable_values(dt):
    # The optional input scan: a clean cube passes; planted non-finite values,
    # non-positive temperatures and negative abundances are counted.
    cube = W.make_cube((6, 7, 40), 2, W.Channels(16, -8.0, 1.0), seed=91, t_dust=True)
    dev = to_device(cube, dt)
    args = (dev["ln_nh2"], dev["t_kin"], dev["v_los"], dev["x_tracer"], dev["t_dust"])
    say(f"[check] field scan {dt}")
    assert rt.iris_rt_check_fields(*args, axis=2, cell_cm=cube.cell_cm) == 0
    dev["ln_nh2"].view(-1)[5] = float("nan")
    dev["v_los"].view(-1)[17] = float("inf")
    dev["t_kin"].view(-1)[3] = 0.0
    dev["t_kin"].view(-1)[9] = -4.0
    dev["t_dust"].view(-1)[100] = float("-inf")
    dev["x_tracer"].view(-1)[11] = -1e-6
    with pytest.raises(rt.IrisError) as e:
        rt.iris_rt_check_fields(*args, axis=2, cell_cm=cube.cell_cm)
    assert e.value.status == 5 and "6 field values" in str(e.value)


@pytest.mark.parametrize("groups", [1, 2, 4])
@pytest.mark.parametrize("scale", [1.0, 40.0])
def test_faint_and_deep_groups_of_cells(scale, groups, monkeypatch):
    # Line depths on both sides of the faint step's bound within groups of four
    # cells, chunk remainders, with a dust temperature field and without; at
    # 40 times the abundance most groups are deep.
    monkeypatch.setenv("IRIS_RT_SIGHTLINES_PER_WAVE", str(groups))
    for t_dust in (False, True):
        cube = W.make_cube((3, 7, 85), 2, W.Channels(70, -17.5, 0.5), seed=80, v_rms_kms=5.0,
                           t_dust=t_dust)
        cube.x_tracer[...] *= scale
        say(f"[fwd] faint and deep groups, scale {scale}, G = {groups}, t_dust {t_dust}")
        dev = to_device(cube, "f32")
        res = gpu_forward(cube, dev)
        ref = oracle.forward(problem(cube, dequantised(dev)), W.LINE_13CO_21)
        for k in "TCDLB":
            e = M.err_inf(res[k].double().cpu().numpy(), ref[k])
            assert e <= TOL_FWD, (k, e)


def test_temperatures_outside_the_tables():
    # Below 1 K and above 65536 K the level and source functions are direct.
    cube = W.make_cube((2, 5, 70), 2, W.Channels(64, -16.0, 0.5), seed=81, v_rms_kms=4.0)
    t = np.geomspace(0.3, 3e5, cube.t_kin.size).reshape(cube.t_kin.shape)
    cube.t_kin[...] = t
    say("[fwd] temperatures from 0.3 to 3e5 K")
    dev = to_device(cube, "f32")
    line = line_dict(t_inf_k=1e6)
    res = gpu_forward(cube, dev, line)
    ref = oracle.forward(problem(cube, dequantised(dev)), line)
    for k in "TCDLB":
        e = M.err_inf(res[k].double().cpu().numpy(), ref[k])
        assert e <= TOL_FWD, (k, e)


@pytest.mark.parametrize("mode", [("formal", "thick"), ("smooth", "thick"), ("formal", "thin")])
@pytest.mark.parametrize("field", ["t_kin", "t_dust"])
def test_cold_cells(field, mode):
    # Down to a thousandth of a kelvin, where e^{T0/T} overflows: no emission.
    cube = W.make_cube((2, 5, 70), 2, W.Channels(64, -16.0, 0.5), seed=82, v_rms_kms=4.0,
                       t_dust=field == "t_dust")
    t = getattr(cube, field).reshape(-1)
    t[::5] = np.geomspace(1e-3, 0.3, t[::5].size)
    say(f"[fwd] cold {field}, {mode}")
    dev = to_device(cube, "f32")
    line = line_dict(integrator=mode[0], transfer=mode[1])
    res = gpu_forward(cube, dev, line)
    ref = oracle.forward(problem(cube, dequantised(dev)), line)
    for k in "TCDLB":
        e = M.err_inf(res[k].double().cpu().numpy(), ref[k])
        assert e <= TOL_FWD, (k, e)


@pytest.mark.parametrize("axis,n", [(1, 8190), (0, 8200), (1, 8200), (2, 8200)])
def test_fields_around_four_gigabytes(axis, n):
    # FP64 fields just below and above 2^32 bytes, where the march's field
    # offsets go from 32 to 64 bits: the last sightlines against the same ones
    # in a cube of their own, bit for bit, with dust that cuts the march's chunks
    # and under optically thin and selectively thin transfer.
    shape = {0: (64, n, 1024), 1: (n, 64, 1024), 2: (n, 1024, 64)}[axis]
    wide = 64 * n * 1024 * 8 >= 1 << 32
    assert wide == (n == 8200)
    last = {0: np.s_[:, -4:], 1: np.s_[-4:], 2: np.s_[-4:]}[axis]
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    small, big = [], []
    for lo, hi in ((4.0, 9.0), (15.0, 80.0), (-6.0, 6.0), (1e-7, 3e-6)):
        big.append(torch.full(shape, 0.5 * (lo + hi), device="cuda", dtype=torch.float64))
        part = big[-1][last]
        part.copy_(lo + (hi - lo) * torch.rand(part.shape, device="cuda", dtype=torch.float64,
                                               generator=g))
        small.append(part.contiguous())
    for kw in (dict(), dict(kappa_dust_cm2g=3e4), dict(transfer="thin"), dict(transfer="selective")):
        say(f"[fwd] {shape} along {axis}, {kw}")
        args = dict(axis=axis, cell_cm=3e17, channels=rt.Channels(12, -6.0, 1.0),
                    line=line_dict(**kw), components="TL")
        a = rt.iris_rt_forward(*big, **args)
        b = rt.iris_rt_forward(*small, **args)
        torch.cuda.synchronize()
        for k in "TL":
            assert torch.equal(a[k][-4 * 1024:], b[k]), (kw, k)
        del a, b

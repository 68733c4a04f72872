"""Which dedispersion kernel an execute runs, as it reports it: the shapes that
the split kernel is tested at reach it and their hinted plans do not, and the
rules of its use hold on both sides of each of their lines."""
import numpy as np
import pytest
import torch

from paper_1307_5700_amd import synth

from gpu_util import api, to_dev

pytestmark = pytest.mark.gpu

NP = {"f32": np.float32, "f16": np.float16, "u8": np.uint8}


def _plan(C, nd, dtype="f32", dm_step=0.2, dm_start=0.0, tsamp=100e-6, hint=0):
    f0, df = synth.band(C)
    return api().Plan(C, f0, df, tsamp, nd, dm_start, dm_step, dtype=dtype, tile_hint=hint)


def _input(C, T, dtype, ld=None, seed=3):
    rng = np.random.default_rng(seed)
    x = np.clip(100.0 + 20.0 * rng.standard_normal((C, T)), 0, 255).astype(NP[dtype])
    return to_dev(x, ld or (T + 7) // 8 * 8 + 4)             # rows the integer kernels do not take


@pytest.mark.parametrize("rfi", [False, True])
@pytest.mark.parametrize("C,nd,T,dtype,kw", [
    (65, 1, 1200, "f32", {}), (96, 8, 2048, "f16", {}), (131, 9, 2052, "u8", {}),
    (256, 64, 4096, "f32", dict(dm_step=1.0)), (300, 37, 5000, "f16", dict(dm_step=0.7)), (512, 17, 3000, "u8", {}),
    (513, 24, 2600, "f32", {}), (1024, 16, 4004, "f32", dict(dm_start=30.0)),
    (1100, 12, 4000, "u8", dict(dm_start=30.0))])
def test_small_launches_split_unless_hinted(C, nd, T, dtype, kw, rfi):
    A = api()
    plan = _plan(C, nd, dtype, **kw)
    tiled = _plan(C, nd, dtype, hint=plan.tiling["index"], **kw)
    x = _input(C, 2 * T // 8 * 8, dtype)
    for p, name in ((plan, "split"), (tiled, "tiled")):
        state = p.rfi_threshold(x[:, :T]) if rfi else None
        p.execute(x[:, :T], rfi_state=state)
        assert p.last_kernels == (name,)
        beam, n = A.Beam(p), T // 32 * 16           # chunks from 16-byte aligned addresses
        for k in range(3):                                   # with ring samples too
            _, _, nout, _ = p.execute(x[:, k * n:(k + 1) * n], beam=beam)
            assert p.last_kernels == ((name,) if nout else ())


def test_split_needs_more_than_two_channel_groups():
    for C, name in ((64, "tiled"), (65, "split")):
        p = _plan(C, 16)
        p.execute(_input(C, 2048, "f32"))
        assert p.last_kernels == (name,)


@pytest.mark.parametrize("span", [253, 254])
def test_split_rows_hold_a_spread_of_253_samples(span):
    """The widest spread of eight DMs that a staged row holds, and one more:
    equal to the tiled kernel either way."""
    f0, df = synth.band(96)
    f = f0 + df * np.arange(96)
    per_dm = 4150.0 * (1 / f[0] ** 2 - 1 / f[-1] ** 2) / 100e-6
    kw = dict(dm_step=span / 7 / per_dm)
    plan = _plan(96, 8, **kw)
    d = plan.delays()
    assert int((d[7] - d[0]).max()) == span
    tiled = _plan(96, 8, hint=plan.tiling["index"], **kw)
    x = _input(96, 3001, "f32")
    outs = [p.execute(x)[0][:, :3001 - span].clone() for p in (plan, tiled)]
    assert plan.last_kernels == ("split" if span == 253 else "tiled",)
    assert tiled.last_kernels == ("tiled",)
    assert torch.equal(*outs)


def test_split_takes_at_most_four_tiles_a_unit():
    units = torch.cuda.get_device_properties(0).multi_processor_count
    p = _plan(96, 64, tsamp=400e-6)                          # eight blocks of eight DMs
    assert p.tiling["dm_block"] == 48 and units % 2 == 0
    for extra, name in ((0, "split"), (1, "tiled")):
        p.execute(_input(96, 256 * units // 2 + extra + p.max_delay, "f32"))
        assert p.last_kernels == (name,)


@pytest.mark.parametrize("C,nd,T,dtype,ring,name", [
    (865, 11, 107108, "f32", False, "tiled"), (865, 11, 90000, "f32", False, "split"),   # 3.3 and 2.8 tiles a unit
    (132, 12, 76106, "f32", False, "tiled"), (132, 12, 60000, "f32", False, "split"),    # 2.3, 1.8
    (73, 96, 11264, "u8", True, "tiled"), (73, 96, 4096, "u8", True, "split"),           # 2.1, 0.8
    (100, 96, 11264, "u8", True, "split"),
], ids=str)
def test_split_takes_fewer_tiles_of_few_dms_or_channels(C, nd, T, dtype, ring, name):
    """Rows staged once per eight DMs, and workgroups of three waves, pay less
    (on a GPU of 256 units)."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("sizes chosen for 256 compute units")
    A = api()
    p = _plan(C, nd, dtype, tsamp=400e-6)
    x = _input(C, T + (0 if ring else p.max_delay), dtype)
    beam = A.Beam(p) if ring else None
    state = p.rfi_threshold(x) if ring else None             # cleaned: float kernels
    for _ in range(3 if ring else 1):
        p.execute(x, rfi_state=state, beam=beam)
    assert p.last_kernels == (name,)


def test_8_bit_chunks_report_their_kernels():
    A = api()
    plan, packed = _plan(512, 96, "u8"), _plan(512, 96, "u8", hint=1)
    x = _input(512, 8192, "u8", ld=8192)
    for p, name in ((plan, "matrix8"), (packed, "packed8")):
        p.execute(x)
        assert p.last_kernels == (name,) and p.last_integer_kernel
        p.execute(x, rfi_state=p.rfi_threshold(x))
        assert p.last_kernels in (("tiled",), ("split",)) and not p.last_integer_kernel
        beam = A.Beam(p)
        for k in range(2):
            p.execute(x[:, 4096 * k:4096 * (k + 1)], beam=beam)
            assert p.last_kernels[-1] == name and len(p.last_kernels) == 1 + k
    wide = _plan(16, 33, "u8", tsamp=51.2e-6)                # too many shifts for the one-hot table
    wide.execute(_input(16, 2048, "u8", ld=2048))
    assert wide.last_kernels == ("packed8",)


@pytest.mark.parametrize("C,nd,T,name", [(13, 1, 1143, "packed8"), (20, 505, 6000, "packed8"), (66, 3, 1346, "packed8"),
                                         (93, 19, 9081, "matrix8"), (300, 64, 9000, "matrix8")])
def test_few_channels_take_the_packed_add_kernel(C, nd, T, name):
    """Equal delays (every DM fits the one-hot table): the channels decide, and
    either kernel gives the packed-add kernel's bits."""
    plan, packed = [_plan(C, nd, "u8", dm_step=0.0, hint=h) for h in (0, 1)]
    x = _input(C, T, "u8", ld=(T + 7) // 8 * 8)
    outs = [p.execute(x)[0][:, :T].clone() for p in (plan, packed)]
    assert plan.last_kernels == (name,) and packed.last_kernels == ("packed8",)
    assert torch.equal(*outs)

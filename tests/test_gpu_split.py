"""Launches of fewer tiles than the GPU has compute units split their channel
groups over waves: every output equals the tiled kernel's bits (a tile_hint
plan never takes the split kernel), single shot and streamed, with and without
cleaning, at the edges of its DM blocks, time tiles, groups and rounds."""
import numpy as np
import pytest
import torch

from paper_1307_5700_amd import synth

from gpu_util import api, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(C=65, nd=1, T=1200, dtype="f32"),                   # three groups, the last of one channel; one DM
    dict(C=96, nd=8, T=2048, dtype="f16"),                   # whole groups, one whole DM block
    dict(C=131, nd=9, T=2052, dtype="u8"),                   # a DM block of one DM
    dict(C=256, nd=64, T=4096, dtype="f32", dm_step=1.0),    # wide delay spread in a DM block
    dict(C=300, nd=37, T=5000, dtype="f16", dm_step=0.7),    # ragged
    dict(C=512, nd=17, T=3000, dtype="u8"),                  # sixteen groups: one round of sixteen waves
    dict(C=513, nd=24, T=2600, dtype="f32"),                 # seventeen: two rounds of nine
    dict(C=1024, nd=16, T=4004, dtype="f32", dm_start=30.0),
    dict(C=1100, nd=12, T=4000, dtype="u8", dm_start=30.0),  # three rounds
], ids=lambda k: "-".join(f"{n}{v}" for n, v in k.items()))
@pytest.mark.parametrize("rfi", [False, True])
def test_split_equals_tiled(kw, rfi):
    A = api()
    f0, df = synth.band(kw["C"])
    beam = synth.Beam(name="split", nchans=kw["C"], f_ch0_mhz=f0, df_mhz=df, tsamp_s=100e-6, ndms=kw["nd"],
                      dm_start=kw.get("dm_start", 0.0), dm_step=kw.get("dm_step", 0.2), nsamps=kw["T"],
                      dtype=kw["dtype"], seed=kw["C"])
    T = kw["T"]
    rng = np.random.default_rng(kw["C"] + kw["nd"])
    x = 100.0 + 20.0 * rng.standard_normal((kw["C"], 2 * T))
    x[:, 300:306] += 90.0                                    # spectra and chunks for the cleaning to flag
    x[5, 512:1100] += 100.0
    x = np.clip(x, 0, 255).astype({"f32": np.float32, "f16": np.float16, "u8": np.uint8}[kw["dtype"]])
    plan = A.Plan.from_beam(beam)
    tiled = A.Plan.from_beam(beam, tile_hint=plan.tiling["index"])
    outs = []
    for p in (plan, tiled):
        got = []
        xd = to_dev(x[:, :T], (T + 7) // 8 * 8 + 4)          # rows the integer kernels do not take
        state = p.rfi_threshold(xd) if rfi else None
        out, _, nout, _ = p.execute(xd[:, :T], rfi_state=state)
        got.append(out[:, :nout].clone())
        b = A.Beam(p)
        for lo, n in ((0, 600), (600, 8 * (T // 8)), (600 + 8 * (T // 8), 256)):
            xc = to_dev(x[:, lo:lo + n], (n + 7) // 8 * 8 + 4)
            state = p.rfi_threshold(xc) if rfi else None
            out, _, nout, _ = p.execute(xc[:, :n], rfi_state=state, beam=b)
            got.append(out[:, :nout].clone() if nout else None)
        outs.append(got)
    for a, t in zip(*outs):
        assert (a is None) == (t is None)
        assert a is None or torch.equal(a, t)

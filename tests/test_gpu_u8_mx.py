"""Matrix-core kernel for 8-bit chunks without cleaning: its sums are exact
integers, so every output equals the oracle's sum and the packed-add kernel's
bits, whatever the tile edges, the channel padding or the band's direction."""
import numpy as np
import pytest

import oracle
from paper_1307_5700_amd import synth

from gpu_util import api, to_dev

pytestmark = pytest.mark.gpu


def _beam(C, nd, T, dm_step=0.2, dm_start=0.0, tsamp=51.2e-6, descending=False):
    f0, df = synth.band(C)
    if descending:
        f0, df = f0 + (C - 1) * df, -df
    return synth.Beam(name="mx", nchans=C, f_ch0_mhz=f0, df_mhz=df, tsamp_s=tsamp, ndms=nd, dm_start=dm_start,
                      dm_step=dm_step, nsamps=T, dtype="u8", seed=C + nd)


@pytest.mark.parametrize("kw", [
    dict(C=1, nd=1, T=64),                                   # one channel, one DM, one partial tile
    dict(C=16, nd=33, T=2048),                               # one cell; a DM block of one DM
    dict(C=129, nd=32, T=2048),                              # one channel past a partial sum; whole DM blocks
    dict(C=128, nd=31, T=1600, dm_step=0.1),                 # a partial sum without padding
    dict(C=300, nd=48, T=4001, tsamp=100e-6),                # odd length
    dict(C=1024, nd=40, T=9000, dm_start=100.0),             # many shifts per step (8 and more)
    dict(C=1024, nd=35, T=8192, descending=True, dm_start=60.0),
    dict(C=200, nd=64, T=3000, dm_step=0.0, dm_start=20.0),  # every DM the same delays
    dict(C=2048, nd=20, T=6000, dm_start=40.0),              # more channels per partial sum
    dict(C=700, nd=33, T=8000, dm_step=0.45, dm_start=30.0), # near the widest spread that fits the tile
], ids=lambda k: "-".join(f"{n}{v}" for n, v in k.items()))
def test_equals_oracle_and_packed_add_kernel(kw):
    A = api()
    beam = _beam(**kw)
    s = oracle.delay_table(**beam.plan_kwargs())
    rng = np.random.default_rng(beam.seed)
    T = beam.nsamps
    x = rng.integers(0, 256, (beam.nchans, T), dtype=np.uint8)
    x[:, : T // 8] = 255                                     # saturated, and blanked, stretches
    x[:, T // 8: T // 4] = 0
    xd = to_dev(x, (T + 7) // 8 * 8)
    ref = oracle.dedisperse(x, s).astype(np.float32)
    for hint in (0, 1):
        try:
            plan = A.Plan.from_beam(beam, tile_hint=hint)
        except A.L.MbError:
            assert hint == 1                                 # the widest spreads do not fit that tiling
            continue
        out, _, nout, _ = plan.execute(xd)
        assert plan.last_integer_kernel and nout == ref.shape[1]
        assert np.array_equal(out[:, :nout].cpu().numpy(), ref), hint

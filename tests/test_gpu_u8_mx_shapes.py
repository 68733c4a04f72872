"""The matrix-core kernel at the edges of its tables, each shape asserted to run
on it: several partial sums of 1, 2, 4 and 8 steps, ragged last ones, 9 to 16
shifts (the second half of the one-hot table), tiles below 512 outputs, DM
blocks of one DM, and the first plan past its shifts.  Every output equals the
oracle's sum and the packed-add kernel's bits."""
import numpy as np
import pytest

import oracle
from paper_1307_5700_amd import synth

from gpu_util import api, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    # steps of a partial sum, most shifts, outputs of a tile
    dict(C=1025, nd=33, step=0.47),                          # 1, 13, 320: 17 sums, the last of one channel
    dict(C=513, nd=48, step=0.3, d0=30.0),                   # 1, 16, 452
    dict(C=129, nd=40, step=0.29, d0=30.0, tsamp=200e-6),    # 1, 16, 512: 3 sums, the last of one channel
    dict(C=640, nd=48, step=0.34, d0=30.0, tsamp=100e-6),    # 2, 16, 512: 5 sums
    dict(C=640, nd=48, step=0.36, d0=30.0, tsamp=100e-6),    # 2 would need 17: 1, 10, 512
    dict(C=1024, nd=48, step=0.28, descending=True),         # 2, 16, 464
    dict(C=1300, nd=64, step=0.09),                          # 2, 6, 512: 11 sums, the last of 20 channels
    dict(C=1000, nd=33, step=0.09, d0=30.0, tsamp=200e-6),   # 4, 5, 512: 4 sums, padded
    dict(C=1000, nd=48, step=0.03, tsamp=200e-6),            # 8, 4, 512: 2 sums, padded
    dict(C=300, nd=33, step=0.34, tsamp=100e-6, packed=True),  # 1, 17: one shift too many
], ids=lambda k: "-".join(f"{n}{v}" for n, v in k.items()))
def test_equals_oracle_and_packed_add_kernel(kw):
    A = api()
    C, tsamp = kw["C"], kw.get("tsamp", 51.2e-6)
    f0, df = synth.band(C)
    if kw.get("descending"):
        f0, df = f0 + (C - 1) * df, -df
    args = dict(nchans=C, f_ch0_mhz=f0, df_mhz=df, tsamp_s=tsamp, ndms=kw["nd"], dm_start=kw.get("d0", 0.0),
                dm_step=kw["step"])
    s = oracle.delay_table(**args)
    T = int(s.max()) + 1301                                  # three or more tiles, the last partial
    x = np.random.default_rng(C).integers(0, 256, (C, T), dtype=np.uint8)
    x[:, : T // 8] = 255                                     # saturated, and blanked, stretches
    x[:, T // 8: T // 4] = 0
    xd = to_dev(x, (T + 7) // 8 * 8)
    ref = oracle.dedisperse(x, s).astype(np.float32)
    plan = A.Plan(dtype="u8", **args)
    packed = A.Plan(dtype="u8", tile_hint=plan.tiling["index"], **args)
    for p, kernel in ((plan, "packed8" if kw.get("packed") else "matrix8"), (packed, "packed8")):
        out, _, nout, _ = p.execute(xd)
        assert p.last_kernels == (kernel,) and nout == ref.shape[1]
        assert np.array_equal(out[:, :nout].cpu().numpy(), ref), kernel

"""The packed-add kernel at the sizes that its 16-bit partial sums, offset
outputs and captured launches are for, asserted to run: plans with a tile_hint
take it where others take the matrix-core kernel."""
import numpy as np
import pytest
import torch

import oracle
from paper_1307_5700_amd import synth

from gpu_util import api, to_dev

pytestmark = pytest.mark.gpu


def _packed(C, nd, T):
    f0, df = synth.band(C)
    b = synth.Beam(name=f"packed{C}", nchans=C, f_ch0_mhz=f0, df_mhz=df, tsamp_s=51.2e-6, ndms=nd, dm_start=0.0,
                   dm_step=0.2, nsamps=T, dtype="u8", seed=5)
    b.pulses = [synth.Pulse(dm_index=nd // 2, t0=T // 3, width=4, amp=1.0)]
    s = oracle.delay_table(**b.plan_kwargs())
    return api().Plan.from_beam(b, tile_hint=1), s, synth.render(b, s)


def _run(plan, x):
    out, _, nout, _ = plan.execute(to_dev(x, (x.shape[1] + 7) // 8 * 8))
    assert plan.last_kernels == ("packed8",)
    return out[:, :nout].cpu().numpy()


@pytest.mark.parametrize("C,nd,T", [(1024, 97, 16384), (517, 48, 9000), (2048, 130, 20000), (333, 51, 8195),
                                    (8192, 48, 4096)])
def test_equals_oracle(C, nd, T):
    """Partial sums widened every 256 channels, up to 32 times, remainders of
    256 and 4 channels, partial DM blocks and tiles; all-255 input, where every
    partial reaches 65280."""
    plan, s, x = _packed(C, nd, T)
    assert np.array_equal(_run(plan, x), oracle.dedisperse(x, s).astype(np.float32))
    assert np.all(_run(plan, np.full((C, T), 255, np.uint8)) == np.float32(C * 255))


def test_streamed_chunks_equal_single_shot():
    """Outputs of the chunk alone go to an offset behind those that reach into
    the ring."""
    A = api()
    plan, s, x = _packed(512, 96, 3 * 4096)
    beam, outs = A.Beam(plan), []
    for k in range(3):
        out, _, nout, _ = plan.execute(to_dev(x[:, k * 4096:(k + 1) * 4096], 4096), beam=beam)
        assert plan.last_kernels == (("packed8",) if k == 0 else ("tiled", "packed8"))
        outs.append(out[:, :nout].cpu().numpy())
    assert np.array_equal(np.concatenate(outs, axis=1), _run(plan, x))


def test_captured_step_replays_exactly():
    A = api()
    T = 8192
    plan, s, x = _packed(512, 96, 3 * T)
    xbuf = torch.zeros((512, T), dtype=torch.uint8, device="cuda")
    xbuf.copy_(torch.from_numpy(np.ascontiguousarray(x[:, :T])))
    g = A.ChunkGraph(plan, xbuf, rfi=False, nsigma=6.0)
    for k in range(3):
        chunk = np.ascontiguousarray(x[:, k * T:(k + 1) * T])
        xbuf.copy_(torch.from_numpy(chunk))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        want = _run(plan, chunk)
        assert np.array_equal(g.out[:, :g.nout].cpu().numpy(), want), k
        assert np.array_equal(want, oracle.dedisperse(chunk, s).astype(np.float32)), k


def test_paper_beam_at_full_size():
    """1024 channels x 65536 samples x 640 DMs: sampled rows equal the oracle's
    sums, the whole plane the matrix-core kernel's."""
    A = api()
    b = synth.paper_beam(dtype="u8")
    plan, default = A.Plan.from_beam(b, tile_hint=1), A.Plan.from_beam(b)
    s = plan.delays()
    x = synth.render(b, s)
    D = _run(plan, x)
    rows = np.array([0, 1, 47, 48, 320, 639])
    assert np.array_equal(D[rows].astype(np.float64), oracle.dedisperse_rows(x, s, rows, D.shape[1]))
    out, _, nout, _ = default.execute(to_dev(x, (x.shape[1] + 7) // 8 * 8))
    assert default.last_kernels == ("matrix8",)
    assert np.array_equal(out[:, :nout].cpu().numpy(), D)

"""The matrix-core kernel's rules, compiled for the CPU: how many steps share a
partial sum, and which launches it takes from the packed-add kernel."""
import subprocess

import numpy as np
import pytest

import oracle
from paper_1307_5700_amd import synth

HERE = __file__.rsplit("/", 1)[0]

PROG = r"""
#include <cstdio>
#include <vector>
#include "mx_rule.h"
int main(int argc, char**) {
  int C, N;
  if (argc > 1) {
    long long nout;
    int ns;
    while (std::scanf("%d %d %lld %d", &C, &N, &nout, &ns) == 4)
      std::printf("%d\n", mbtp::mx_pays(C, N, nout, ns, 32, 512, 48, 512, 256));
    return 0;
  }
  while (std::scanf("%d %d", &N, &C) == 2) {
    std::vector<int32_t> d((size_t)N * C);
    for (auto& v : d) if (std::scanf("%d", &v) != 1) return 1;
    const double s = mbtp::mx_spread(d.data(), N, C);
    const int ns = mbtp::mx_steps(s, C);
    std::printf("%.17g %d %d\n", s, ns, mbtp::mx_padded_steps(C, ns));
  }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("mx_rule")
    (d / "p.cpp").write_text(PROG)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", HERE + "/../paper_1307_5700_amd/csrc", str(d / "p.cpp"), "-o",
                    str(d / "p")], check=True, capture_output=True)

    def pays(launches):
        text = "\n".join(" ".join(map(str, v)) for v in launches)
        out = subprocess.run([str(d / "p"), "pays"], input=text, capture_output=True, text=True, check=True).stdout
        return [v == "1" for v in out.split()]

    def ask(tables):
        text = "\n".join(f"{t.shape[0]} {t.shape[1]} " + " ".join(map(str, t.ravel())) for t in tables)
        out = subprocess.run([str(d / "p")], input=text, capture_output=True, text=True, check=True).stdout
        return [(float(a), int(b), int(c)) for a, b, c in (line.split() for line in out.splitlines())]
    ask.pays = pays
    return ask


def test_padding_is_paid_only_where_it_pays(rule):
    """Channels are padded to whole partial sums: with delays that do not
    spread, the longest partial sums save at most 29.1 / 24.8 of a step's cost
    over single steps, so no more padded steps than that are ever taken."""
    chans = [1, 5, 13, 20, 63, 64, 65, 91, 128, 129, 182, 300, 512, 513, 847, 1024, 1130, 2048, 2049, 4095, 4096]
    for C, (s, ns, steps) in zip(chans, rule([np.zeros((2, C), int) for C in chans])):
        need = -(-C // 64)
        assert s == 0.0 and need <= steps <= need * 29.1 / 24.8, (C, ns, steps)


@pytest.mark.parametrize("C,nd,step", [(1024, 40, 0.2), (200, 64, 0.0), (1024, 1, 0.2), (300, 97, 0.05)])
def test_spread_does_not_depend_on_the_first_dm(rule, C, nd, step):
    """A DM range from 100 spreads as one from 0 (to the rounding of each
    delay), and takes the same steps."""
    f0, df = synth.band(C)
    low, high = [oracle.delay_table(nchans=C, f_ch0_mhz=f0, df_mhz=df, tsamp_s=51.2e-6, ndms=nd, dm_start=d0,
                                    dm_step=step) for d0 in (0.0, 100.0)]
    (s0, n0, _), (s1, n1, _) = rule([np.asarray(low), np.asarray(high)])
    assert abs(s0 - s1) <= 16.0 / max(nd - 1, 1) / C and n0 == n1


def test_few_channels_stay_with_the_packed_add_kernel(rule):
    """A step costs the matrix-core kernel the same whatever it holds, so
    launches of a few channels are the packed-add kernel's, for any DMs and
    outputs, and launches of full steps are not."""
    sizes = [(nd, nout) for nd in (1, 5, 32, 33, 48, 49, 640, 65535) for nout in (1, 511, 513, 9000, 60000, 1 << 24)]
    assert not any(rule.pays([(C, nd, nout, 1) for C in (1, 8, 16) for nd, nout in sizes]))
    assert all(rule.pays([(C, nd, nout, 1) for C in (128, 192, 1024, 4096) for nd, nout in sizes]))

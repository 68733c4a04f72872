"""Which launches the split kernel takes, compiled for the CPU: its choice at
measured pairs of times (us, split and tiled) on 256 compute units, and the
limits that hold for every launch."""
import subprocess

import pytest

HERE = __file__.rsplit("/", 1)[0]

PROG = r"""
#include <cstdio>
#include "split_rule.h"
int main() {
  int C, nd, bytes, ring, bd, bt;
  long long nout;
  while (std::scanf("%d %d %lld %d %d %d %d", &C, &nd, &nout, &bytes, &ring, &bd, &bt) == 7) {
    const long long tiles = (nd + bd - 1) / bd * ((nout + bt - 1) / bt), split = (nd + 7) / 8 * ((nout + 255) / 256);
    std::printf("%d\n", mbtp::split_pays(C, nd, bytes, ring != 0, bd, tiles, split, 256));
  }
}
"""


@pytest.fixture(scope="module")
def pays(tmp_path_factory):
    d = tmp_path_factory.mktemp("split_rule")
    (d / "p.cpp").write_text(PROG)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", HERE + "/../paper_1307_5700_amd/csrc", str(d / "p.cpp"), "-o",
                    str(d / "p")], check=True, capture_output=True)

    def ask(launches):
        text = "\n".join(" ".join(map(str, v)) for v in launches)
        out = subprocess.run([str(d / "p")], input=text, capture_output=True, text=True, check=True).stdout
        return [v == "1" for v in out.split()]
    return ask


# channels, DMs, outputs, bytes a sample, ring, tile; us split, us tiled
MEASURED = [
    ((865, 11, 107084, 4, 0, 48, 512), 229.2, 188.8), ((73, 214, 5464, 1, 1, 48, 512), 43.6, 36.8),
    ((71, 15, 100916, 4, 0, 48, 512), 30.6, 27.1), ((139, 11, 113157, 4, 0, 48, 512), 55.4, 47.1),
    ((1607, 16, 129166, 2, 0, 48, 512), 353.6, 325.7), ((69, 91, 5728, 1, 1, 48, 512), 35.8, 34.0),
    ((94, 12, 97670, 4, 0, 48, 512), 31.4, 30.1), ((132, 12, 76106, 4, 0, 48, 512), 40.2, 36.2),
    ((72, 2, 71501, 4, 0, 48, 512), 20.7, 19.4), ((296, 36, 57885, 4, 0, 48, 512), 103.6, 89.1),
    ((910, 11, 103585, 1, 0, 48, 512), 194.0, 263.0), ((3438, 10, 82649, 2, 0, 48, 512), 511.0, 731.0),
    ((3872, 16, 87447, 4, 0, 48, 512), 781.0, 1150.0), ((2346, 9, 87415, 1, 0, 48, 512), 413.0, 673.0),
    ((256, 64, 6656, 4, 0, 48, 512), 19.4, 63.5), ((300, 37, 7500, 4, 0, 48, 512), 21.6, 62.5),
]


def test_choice_at_measured_launches(pays):
    for (launch, split, tiled), got in zip(MEASURED, pays([m[0] for m in MEASURED])):
        assert got == (split < tiled), launch


def test_limits(pays):
    sizes = [(nd, nout) for nd in (1, 8, 9, 32, 33, 64, 400) for nout in (1, 256, 257, 5000, 20000, 70000, 200000)]
    for bytes_ in (1, 2, 4):
        for ring in (0, 1):
            for bd in (48, 32, 8):
                for C in (1, 64, 65, 80, 81, 160, 161, 4096):
                    for (nd, nout), got in zip(sizes, pays([(C, nd, n, bytes_, ring, bd, 512) for nd, n in sizes])):
                        tiles = -(-nd // bd) * -(-nout // 512)
                        split = -(-nd // 8) * -(-nout // 256)
                        most = 256 * (2 if bd < 48 else 3 if ring else 4)
                        assert not got or (C > 64 and tiles <= 256 and split <= most)
                        assert got or C <= 64 or tiles > 256 or split > 256     # one a unit always

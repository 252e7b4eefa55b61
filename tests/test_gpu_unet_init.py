"""Initial parameters of a network (GPU): bit for bit those that std::normal_distribution gives for the same seeds, from
a program compiled here, a fresh distribution for every layer on one std::mt19937_64."""
import math
import shutil
import subprocess

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import unet as U  # noqa: E402

pytestmark = pytest.mark.gpu

SOURCE = """
#include <cstdio>
#include <cstdlib>
#include <random>
int main(int argc, char **argv) {
    std::mt19937_64 rng(std::strtoull(argv[1], nullptr, 10));
    for (int a = 2; a + 1 < argc; a += 2) {
        std::normal_distribution<double> nd(0.0, std::strtod(argv[a], nullptr));
        for (long n = std::strtol(argv[a + 1], nullptr, 10); n > 0; --n) {
            const float v = (float)nd(rng);
            std::fwrite(&v, sizeof(v), 1, stdout);
        }
    }
}
"""


@pytest.mark.parametrize("levels,base,seed", [(1, 16, 0), (3, 16, 7), (2, 48, 2 ** 63 + 5)])
def test_initial_parameters(tmp_path, levels, base, seed):
    if not torch.cuda.is_available() or not shutil.which("g++"):
        pytest.skip("needs a GPU and g++")
    from paper_2609_17636_amd.unet import UNet

    (tmp_path / "n.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-ffp-contract=off", str(tmp_path / "n.cpp"), "-o", str(tmp_path / "n")], check=True)
    args, where, o = [str(seed)], [], 0
    for name, shape in U.unet_param_shapes(levels, base, 4):
        k = int(np.prod(shape)) if shape else 1
        if name.endswith("w"):
            fan = shape[3] * 9 if len(shape) == 4 else 0
            args += [repr(math.sqrt(2.0 / fan) if fan else math.sqrt(1.0 / base)), str(k)]
            where.append((o, k))
        o += k
    drawn = np.frombuffer(subprocess.run([str(tmp_path / "n"), *args], check=True, stdout=subprocess.PIPE).stdout, np.float32)
    want, at = np.zeros(o, np.float32), 0
    for s, k in where:
        want[s:s + k] = drawn[at:at + k]
        at += k
    assert at == drawn.size
    got = UNet(levels=levels, base=base, max_batch=1, height=8, width=8, seed=seed).get_params()
    assert np.array_equal(np.asarray(got, np.float32), want)

"""bench.py names the kernel a streaming call runs; the library's own rule, compiled here, must agree."""
import random

import bench
from tests._util import few_row_tiles


def test_bench_names_the_kernel_that_runs():
    rng = random.Random(1)
    size = lambda: rng.choice([128, 512, 768, 1024, 2048, 3072, 4096, 7168, 8064, 8192, 8320, 128 * rng.randint(1, 70)])
    cases = [(rng.randint(1, 300), size(), size(), rng.randint(0, 3), rng.randint(0, 1)) for _ in range(5000)]
    cases += [(T, H, I, w, d) for T in (3, 4, 6, 7, 16, 17, 32, 33, 64, 65, 95, 96, 255, 256) for H in (2048, 4096, 7168, 8192)
              for I in (768, 2048, 4096, 8192, 8320) for w in range(4) for d in (0, 1)]
    for c, ran in zip(cases, few_row_tiles(cases), strict=True):
        assert bench.few_row_tiles(*c) == ran, c

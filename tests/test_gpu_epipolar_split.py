"""The epipolar check where its split over wavefronts can go wrong: hypotheses
around a workgroup's 64, correspondences around the four wavefronts' shares and
the staged 512, and systems whose pivots tie (lattice points) or vanish."""
import numpy as np
import pytest

from test_gpu_epipolar import check_set, ctx, lk, run, make_set  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu
INTR = (410.0, 395.0, 321.5, 243.25)


@pytest.mark.parametrize("kind", ["scene", "lattice", "line"])
def test_split(lk, ctx, kind):  # noqa: F811
    sets, host = [], []
    for n, h in [(8, 1), (9, 63), (11, 64), (66, 65), (511, 5), (512, 130), (513, 64), (515, 3), (1027, 70)]:
        rng = np.random.default_rng(100 * n + h)
        if kind == "scene":
            x = rng.uniform([-2, -2, 4], [2, 2, 9], (n, 3))
            y = x + [0.3, 0.05, 0.1]
            p = x[:, :2] / x[:, 2:] * INTR[:2] + INTR[2:]
            q = y[:, :2] / y[:, 2:] * INTR[:2] + INTR[2:] + rng.normal(0, 0.3, (n, 2))
        elif kind == "lattice":
            p = np.stack([np.arange(n) % 31, np.arange(n) // 31], 1) * 16.0
            q = p + rng.integers(-2, 3, (n, 2))
        else:                                  # all on one line: rank below 8
            p = np.stack([np.arange(n) * 3.0, np.full(n, 50.0)], 1)
            q = p + [4.0, 0.0]
        samples = np.stack([rng.choice(n, 8, replace=False) for _ in range(h)]).astype(np.int32)
        p, q = p.astype(np.float32), q.astype(np.float32)
        sets.append(make_set(p, q, samples, INTR))
        host.append((p, q, samples))
    print(kind, flush=True)
    for d, g, (p, q, samples) in zip(sets, run(lk, ctx, sets), host):
        if kind == "line":
            assert (g["counts"] == -1).all() and g["best"][0] == -1 and not g["inliers"].any()
        elif kind == "scene":
            check_set(d, g, p, q, samples, INTR)
        else:                                  # near-singular draws: the oracle's solve is not comparable
            c = g["counts"]
            k = int(np.flatnonzero(c == c.max())[0]) if c.max() >= 0 else -1
            assert int(g["best"][0]) == k
            if k >= 0:                         # the model solved again scores as it did
                assert int(g["best"][1]) == c[k] == int(g["inliers"].sum())

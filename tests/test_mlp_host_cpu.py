"""The host's selection forward pass (vectors of eight outputs, padded to
whole vectors) on loaded weights, against a plain NumPy forward pass, at the
sizes of the kernel list where the padding changes and beyond the vector
pass's limit of 64."""
import math

import numpy as np
import pytest


def _write(path, chosen, params):
    with open(path, "w") as f:
        f.write("KTSEL 3\nselectors 1\ndtype 0\nkind 3\n")
        f.write(f"chosen {len(chosen)} " + " ".join(map(str, chosen)) + "\ntree 0\n")
        f.write(f"mlp {len(params)}\n" + "\n".join(float(v).hex() for v in params) + "\n")
        f.write("box 0 0 0 0 0 0 0 0 0 0\nend\n")


@pytest.mark.parametrize("k", [1, 2, 7, 8, 9, 31, 32, 33, 64, 65])
def test_host_selection_matches_numpy(kt, tmp_path, k):
    rng = np.random.default_rng(100 + k)
    W1, b1 = rng.normal(size=(64, 6)).astype(np.float32), rng.normal(size=64).astype(np.float32)
    W2, b2 = (rng.normal(size=(64, 64)) / 8).astype(np.float32), rng.normal(size=64).astype(np.float32)
    W3, b3 = (rng.normal(size=(k, 64)) / 8).astype(np.float32), rng.normal(size=k).astype(np.float32)
    chosen = [int(c) for c in rng.permutation(164)[:k]]
    path = str(tmp_path / "sel.txt")
    _write(path, chosen, np.concatenate([a.ravel() for a in (W1, b1, W2, b2, W3, b3)]))
    h = kt.Handle(-1)
    try:
        h.load(path)
        checked = 0
        for _ in range(300):
            M, N, K, b = (int(math.exp(rng.uniform(0, math.log(hi)))) for hi in (5000, 5000, 5000, 64))
            ta, tb = int(rng.integers(2)), int(rng.integers(2))
            x = np.array([math.log2(M) / 12, math.log2(N) / 12, math.log2(K) / 12, math.log2(b) / 6, ta, tb])
            y = np.maximum(np.maximum(x @ W1.T.astype(float) + b1, 0) @ W2.T.astype(float) + b2, 0) \
                @ W3.T.astype(float) + b3
            order = np.sort(y)
            # sums of 64 products of order 1 in FP32: errors below 64 * 2**-23 * 10
            if k > 1 and order[-1] - order[-2] < 1e-4:
                continue
            checked += 1
            assert h.select(M, N, K, b, ta, tb) == chosen[int(y.argmax())]
        assert checked > 200
    finally:
        h.close()

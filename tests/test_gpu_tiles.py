"""Tile-image kernels (full-precision nets with hidden layers) against the
oracle at the edges of their tiles: every number of batch tiles, one and two
unit tiles per workgroup (two from 256 workgroups up), odd unit-tile counts,
fewer input blocks than waves, a short last batch, ragged prediction rows."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu

CASES = [
    # dims, batch, P
    ([40, 33, 3], 20, 3), ([40, 33, 3], 50, 3), ([100, 96, 7], 96, 3), ([100, 96, 7], 128, 3),
    ([40, 33, 3], 150, 3), ([100, 64, 32], 180, 3), ([40, 96, 3], 220, 3), ([300, 64, 10], 256, 3),
    ([20, 30, 2], 7, 2),                      # one input block: three waves have none
    ([70, 64, 5], 20, 256), ([200, 64, 10], 128, 256), ([70, 64, 5], 210, 256),   # two unit tiles per workgroup
    ([200, 70, 40, 10], 50, 4), ([130, 64, 160, 6], 128, 60),                    # three layers
]


@pytest.mark.parametrize("dims,batch,P", CASES)
def test_three_steps_and_prediction_match_the_oracle(dims, batch, P):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2310_10211_amd as g
    n_train, n_test = 2 * batch + max(1, batch // 3), 300
    cfg = synthetic.config(2, P=P, dims=dims, batch=batch, lr=(0.05, 0.2))
    data = synthetic.dataset(cfg, n_train, n_test)
    for k in ("x_train", "x_test"):
        data[k] = np.ascontiguousarray(data[k][:, :dims[0]])
    for k in ("y_train", "y_test"):
        data[k] = data[k] % dims[-1]
    print(f"[gpu] tiles dims={dims} batch={batch} P={P}", flush=True)
    pop = g.Population(cfg, data["x_train"], data["y_train"], data["x_test"], data["y_test"])
    pop.train_epoch(0)
    pop.predict()
    s = pop.scores()
    sample = sorted({0, 1, P - 1})
    ref = oracle.evaluate(cfg, data, variants=sample, epochs=1, mode="f32")
    perm = oracle.permutation(cfg["seed"], 0, n_train)
    init = oracle.population(cfg, sample)
    for v in sample:
        # fp32 sums of at most about 600 terms: 600 2^-24 = 4e-5 of the summed
        # magnitudes at the very worst, 1e-6 in practice, on updates that are a
        # tenth of the weights at most
        p = init[v]["params"].copy()
        oracle.train_steps("f32", dims, p, init[v]["mask"], init[v]["lr"], data["x_train"], data["y_train"], perm,
                           batch, 0, 3)
        got = pop.export(v)["params"].astype(np.float64)
        for (Wg, bg), (Wr, br) in zip(oracle.unpack(got, dims), oracle.unpack(p, dims)):
            assert np.max(np.abs(Wg - Wr)) <= 1e-5 * max(np.max(np.abs(Wr)), 1e-30)
            assert np.max(np.abs(bg - br)) <= 1e-5 * max(np.max(np.abs(br)), 1e-3)
        assert abs(s["train_loss"][v] - ref[v]["train_loss"][0]) <= 1e-5 * abs(ref[v]["train_loss"][0])
        assert abs(s["test_loss"][v] - ref[v]["test_loss"]) <= 1e-5 * abs(ref[v]["test_loss"])
        assert abs(s["test_acc"][v] - ref[v]["test_acc"]) <= 1.0 / n_test      # a tie within rounding
    pop.close()


# (unit tiles, row tiles) per wave of the prediction kernel: rounds of 256
# workgroups times the products of a wave, one more for the operands
TILES = [(2, 8), (2, 4), (1, 4), (1, 2), (1, 1)]


def _tile(width, rows, P):
    nb, nrt = -(-width // 32), rows // 32

    def cost(t):
        nt, rt = t
        return -(-(-(-nb // (4 * nt)) * -(-nrt // rt) * P) // 256) * (nt * rt + 1)
    return min(TILES, key=cost)


@pytest.mark.parametrize("dims,P,n_test,tiles", [
    ([784, 256, 10], 64, 2300, [(2, 8), (1, 4)]),           # two chunks of rows, the second ragged
    ([100, 224, 10], 64, 4500, [(2, 8), (2, 8), (2, 4)]),   # seven unit tiles on waves of two
    ([100, 256, 10], 128, 250, [(2, 4)]),
    ([100, 160, 7], 100, 400, [(2, 8)]),                    # five
    ([100, 96, 10], 40, 200, [(1, 2)]),
    ([100, 40, 3], 5, 2049, [(1, 2), (1, 1)]),
    ([200, 96, 224, 10], 64, 2048, [(1, 4), (2, 8)]),       # two hidden layers
])
def test_prediction_tiles_match_the_oracle(dims, P, n_test, tiles):
    """fp32 prediction on every tile of the forward kernel, over one to three
    chunks of 2,048 rows."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2310_10211_amd as g
    pad = -(-n_test // 256) * 256
    chunks = [min(2048, pad - c) for c in range(0, pad, 2048)]
    assert [_tile(w, r, P) for r in chunks for w in dims[1:-1]] == tiles
    cfg = synthetic.config(2, P=P, dims=dims, dens=(0.5, 1.0))
    data = synthetic.dataset(cfg, 0, n_test)
    x, y = np.ascontiguousarray(data["x_test"][:, :dims[0]]), data["y_test"] % dims[-1]
    data = dict(x_train=data["x_train"], y_train=data["y_train"], x_test=x, y_test=y)
    print(f"[gpu] prediction tiles dims={dims} P={P} n_test={n_test}", flush=True)
    pop = g.Population(cfg, None, None, x, y)
    pop.predict()
    s = pop.scores()
    pop.close()
    sample = sorted({0, 1, P - 1})
    ref = oracle.evaluate(cfg, data, variants=sample, epochs=0, mode="f32")
    for v in sample:                                         # fp32 sums of at most 800 terms, means of n_test losses
        assert abs(s["test_loss"][v] - ref[v]["test_loss"]) <= 1e-5 * abs(ref[v]["test_loss"]), v
        assert abs(s["test_acc"][v] - ref[v]["test_acc"]) <= 1.0 / n_test, v

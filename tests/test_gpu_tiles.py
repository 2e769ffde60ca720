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

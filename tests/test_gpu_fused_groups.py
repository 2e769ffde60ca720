"""Fused training of 128-unit hidden layers at batches of up to 32 rows (two
groups of waves, each taking every second block of 32 inputs) against the
oracle: one to five input blocks, so that a group has none, one or two of the
last ones, short batches, few and many classes, and a continued run."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch,P", [([20, 100, 3], 32, 2), ([40, 128, 10], 32, 3), ([70, 120, 10], 20, 3),
                                          ([128, 128, 20], 32, 2), ([150, 128, 32], 7, 11), ([784, 128, 10], 32, 40)])
def test_groups_match_the_oracle(dims, batch, P):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2310_10211_amd as g
    cfg = synthetic.config(3, P=P, dims=dims, batch=batch, lr=(0.02, 0.1), dens=(0.5, 1.0))
    n_train = 5 * batch + max(1, batch // 3)
    data = synthetic.dataset(cfg, n_train, 200)
    for k in ("x_train", "x_test"):
        data[k] = np.ascontiguousarray(data[k][:, :dims[0]])
    for k in ("y_train", "y_test"):
        data[k] = data[k] % dims[-1]
    print(f"[gpu] fused groups dims={dims} batch={batch} P={P}", flush=True)
    args = (cfg, data["x_train"], data["y_train"], data["x_test"], data["y_test"])
    pop = g.Population(*args)
    pop.train_epoch(0)
    pop.predict()
    s = pop.scores()
    halves = g.Population(*args)                                 # the same epoch in two calls: the same bits
    halves.train_steps(0, 0, 2)
    halves.train_steps(0, 2, halves.steps_per_epoch)
    sample = sorted({0, 1, P - 1})
    ref = oracle.evaluate(cfg, data, variants=sample, epochs=1, mode="bf16")
    init = oracle.population(cfg, sample)
    perm = oracle.permutation(cfg["seed"], 0, n_train)
    for v in sample:
        e = pop.export(v)
        assert np.array_equal(halves.export(v)["params"], e["params"])
        assert np.array_equal(e["mask"], init[v]["mask"])
        p = init[v]["params"].copy()
        oracle.train_steps("bf16", dims, p, init[v]["mask"], init[v]["lr"], data["x_train"], data["y_train"], perm,
                           batch, 0, 6)
        # the same values are rounded to bf16 (2^-9 relative); sums in another
        # order move single operands by one ulp, and a step moves a weight by
        # at most lr times a gradient: 2^-7 of the distance from the start,
        # over six steps, bounds what those moves can add
        d0 = p.astype(np.float64) - init[v]["params"]
        d = e["params"].astype(np.float64) - init[v]["params"]
        assert np.linalg.norm(d - d0) <= 2.0 ** -7 * np.linalg.norm(d0), v
        assert abs(s["train_loss"][v] - ref[v]["train_loss"][0]) <= 2e-2 * abs(ref[v]["train_loss"][0])
        assert abs(s["test_loss"][v] - ref[v]["test_loss"]) <= 2e-2 * abs(ref[v]["test_loss"])
    pop.close()
    halves.close()

"""bf16 training on the tile-image kernels against the oracle: every number of
batch tiles, one and two unit tiles per workgroup, odd unit-tile counts, fewer
input blocks than waves, short last batches, two and three layers, many
classes; nets that the fused or the streaming kernel would take with more
variants; and narrowed variants."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu

CASES = [
    # dims, batch, P
    ([40, 33, 3], 20, 3), ([40, 33, 3], 50, 3), ([100, 96, 7], 96, 3), ([100, 96, 7], 128, 3),
    ([40, 33, 3], 150, 3), ([100, 64, 32], 180, 3), ([40, 96, 3], 220, 3), ([300, 64, 10], 256, 3),
    ([20, 30, 2], 7, 2),                                             # one input block: three waves have none
    ([70, 64, 5], 20, 256), ([200, 64, 10], 128, 256),               # two unit tiles per workgroup
    ([200, 70, 40, 10], 50, 4), ([130, 64, 160, 6], 100, 60),        # three layers
    ([520, 256, 10], 128, 4), ([600, 100, 10], 100, 5),              # few variants of nets the fused kernel takes
    ([512, 128, 10], 200, 3), ([512, 128, 128, 5], 128, 3),          # and of nets the streaming kernel takes
]


@pytest.mark.parametrize("dims,batch,P", CASES)
def test_bf16_tiles_match_the_oracle(dims, batch, P):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2310_10211_amd as g
    n_train, n_test = 2 * batch + max(1, batch // 3), 300
    cfg = synthetic.config(3, P=P, dims=dims, batch=batch, lr=(0.02, 0.1), dens=(0.5, 1.0))
    data = synthetic.dataset(cfg, n_train, n_test)
    for k in ("x_train", "x_test"):
        data[k] = np.ascontiguousarray(data[k][:, :dims[0]])
    for k in ("y_train", "y_test"):
        data[k] = data[k] % dims[-1]
    print(f"[gpu] bf16 tiles dims={dims} batch={batch} P={P}", flush=True)
    pop = g.Population(cfg, data["x_train"], data["y_train"], data["x_test"], data["y_test"])
    pop.train_epoch(0)
    pop.predict()
    s = pop.scores()
    sample = sorted({0, 1, P - 1})
    ref = oracle.evaluate(cfg, data, variants=sample, epochs=1, mode="bf16")
    perm = oracle.permutation(cfg["seed"], 0, n_train)
    init = oracle.population(cfg, sample)
    for v in sample:
        p = init[v]["params"].copy()
        oracle.train_steps("bf16", dims, p, init[v]["mask"], init[v]["lr"], data["x_train"], data["y_train"], perm,
                           batch, 0, 3)
        # the same values are rounded to bf16 (2^-9 relative); sums in another
        # order move single operands by one ulp: 2^-7 of the distance from the
        # start bounds what those moves can add over three steps
        e = pop.export(v)
        start = init[v]["params"].astype(np.float64)
        d0 = p.astype(np.float64) - start
        assert np.linalg.norm(e["params"].astype(np.float64) - start - d0) <= 2.0 ** -7 * np.linalg.norm(d0), v
        assert np.array_equal(e["mask"], init[v]["mask"])
        assert abs(s["train_loss"][v] - ref[v]["train_loss"][0]) <= 2e-2 * abs(ref[v]["train_loss"][0])
        assert abs(s["test_loss"][v] - ref[v]["test_loss"]) <= 2e-2 * abs(ref[v]["test_loss"])
    # a narrowed variant trains like the oracle's, its neighbours undisturbed
    if len(dims) == 3 and dims[1] > 40:
        pop.set_genomes([[(g.EDIT_WIDTH, 1, 20)] if v == 1 else [] for v in range(P)], 0.05)
        pop.train_epoch(0)
        e = pop.export(1)
        W1 = e["params"][:dims[0] * dims[1]].reshape(dims[0], dims[1])
        assert np.all(W1[:, 20:] == 0) and np.any(W1[:, :20] != 0) and np.all(np.isfinite(pop.scores()["train_loss"]))
    pop.close()

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
    ([60, 160, 7], 60, 64), ([60, 192, 7], 200, 86),                 # five; three pairs, two of them removed
    ([200, 70, 40, 10], 50, 4), ([130, 64, 160, 6], 100, 60),        # three layers
    ([520, 256, 10], 128, 4), ([600, 100, 10], 100, 5),              # few variants of nets the fused kernel takes
    ([512, 128, 10], 200, 3), ([512, 128, 10], 250, 3), ([512, 128, 128, 5], 128, 3),   # and the streaming kernel (not 200 rows)
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
    # a narrowed variant trains like the oracle's, its neighbours like those of
    # a population without it (the workgroups of its removed unit tiles return)
    if len(dims) == 3 and dims[1] > 40:
        runs = []
        for narrow in (True, False):
            pop.set_genomes([[(g.EDIT_WIDTH, 1, 20)] if v == 1 and narrow else [] for v in range(P)], 0.05)
            pop.train_epoch(0)
            runs.append([pop.export(v)["params"] for v in (0, 1, P - 1)])
            assert np.all(np.isfinite(pop.scores()["train_loss"]))
        for i in (0, 2):
            if (0, 1, P - 1)[i] != 1:
                assert runs[0][i].tobytes() == runs[1][i].tobytes(), i
        mask, bmask = oracle.structure_masks(dims, [dims[0], 20, dims[2]], [1, 1], oracle.genome_mask(cfg["seed"], dims, [], []))
        start, _ = oracle.variant_init(cfg["seed"], 0, dims, 1 << 24)
        n1 = dims[0] * dims[1]
        start[:n1] *= mask[:n1]
        start[n1 + dims[1]:n1 + dims[1] + dims[1] * dims[2]] *= mask[n1:]
        p = start.copy()
        oracle.train_steps("bf16", dims, p, mask, 0.05, data["x_train"], data["y_train"], perm, batch, 0, 3, bmask=bmask)
        got = runs[0][1].astype(np.float64)
        assert np.all(got[p == 0] == 0)
        assert np.linalg.norm(got - p) <= 2.0 ** -7 * np.linalg.norm(p - start)
    pop.close()

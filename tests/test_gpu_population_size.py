"""What a population's size changes of a variant's training: the kernel (bf16
nets that the fused or the streaming kernel takes train on the tile kernels
while the population is small) and, on the tile kernels, how many unit tiles
and waves share a workgroup.  Within a range of sizes the bits are the same;
across a line the same values are rounded and summed, in another order.  Each
size is compared with the oracle and the sizes of a range with each other."""
import numpy as np
import pytest

import oracle
import synthetic
from conftest import training_path

pytestmark = pytest.mark.gpu

# ranges of sizes with the same bits.  On the tile kernels the lines are eight
# waves (few row tiles, P * unit tiles <= 256) and two unit tiles a workgroup
# (an even number of them, P * unit tiles / 2 >= 256).
CASES = [
    ([200, 128, 10], 128, "f32", [(3, 60, "tiles"), (128, 130, "tiles")]),
    ([70, 64, 5], 20, "f32", [(3, 128, "tiles"), (129, 255, "tiles"), (256, 257, "tiles")]),   # one row tile: all three
    ([300, 96, 10], 20, "f32", [(3, 85, "tiles"), (86, 90, "tiles")]),                         # an odd number of unit tiles
    ([130, 64, 160, 6], 150, "f32", [(3, 255, "tiles"), (256, 257, "tiles")]),                 # three layers, five row tiles
    ([70, 64, 5], 20, "bf16", [(3, 128, "tiles"), (129, 255, "tiles"), (256, 257, "tiles")]),
    ([300, 192, 10], 100, "bf16", [(3, 42, "tiles"), (43, 85, "tiles"), (86, 87, "tiles")]),   # four row tiles
    ([100, 320, 64, 3], 40, "bf16", [(3, 25, "tiles"), (26, 51, "tiles"), (52, 53, "tiles")]),
    ([200, 64, 10], 200, "bf16", [(3, 255, "tiles"), (256, 257, "tiles")]),                    # seven row tiles
    ([784, 256, 10], 128, "bf16", [(3, 32, "tiles"), (33, 40, "fused")]),
    ([512, 128, 256, 10], 128, "bf16", [(17, 32, "tiles"), (33, 40, "streamed 2")]),
    ([512, 256, 160, 10], 256, "bf16", [(33, 64, "tiles"), (65, 70, "streamed 1")]),
]


@pytest.mark.parametrize("dims,batch,dtype,ranges", CASES)
def test_population_sizes_on_each_side_of_a_line(dims, batch, dtype, ranges):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2310_10211_amd as g
    cfg = synthetic.config(3, dims=dims, batch=batch, dtype=dtype, lr=(0.02, 0.1), dens=(0.5, 1.0))
    n_train = 2 * batch + max(1, batch // 3)
    data = synthetic.dataset(cfg, n_train, 100)
    for k in ("x_train", "x_test"):
        data[k] = np.ascontiguousarray(data[k][:, :dims[0]])
    for k in ("y_train", "y_test"):
        data[k] = data[k] % dims[-1]
    init = oracle.population(cfg, [0, 1, 2])
    perm = oracle.permutation(cfg["seed"], 0, n_train)
    want, loss = {}, {}
    for v in range(3):
        want[v] = init[v]["params"].copy()
        ce, _ = oracle.train_steps(dtype, dims, want[v], init[v]["mask"], init[v]["lr"], data["x_train"],
                                   data["y_train"], perm, batch, 0, 3)
        loss[v] = ce / n_train
    # Bars of the kernels' own tests after three steps: fp32 sums of at most
    # about 800 terms; bf16 operands moved by one ulp, 2^-7 of the distance
    # from the start.
    for small, large, path in ranges:
        got = []
        for P in (small, large):
            print(f"[gpu] population size {P}: dims={dims} batch={batch} dtype={dtype}", flush=True)
            pop = g.Population(dict(cfg, P=P), data["x_train"], data["y_train"], data["x_test"], data["y_test"])
            assert training_path(pop, lambda: pop.train_epoch(0)) == path, P
            s = pop.scores()["train_loss"]
            got.append((s[:3].tobytes(), [pop.export(v)["params"] for v in range(3)]))
            for v in range(3):
                assert abs(s[v] - loss[v]) <= (1e-5 if dtype == "f32" else 2e-2) * abs(loss[v]), (P, v)
            pop.close()
        assert got[0][0] == got[1][0], (small, large)
        for v in range(3):
            a, start = got[0][1][v].astype(np.float64), init[v]["params"]
            assert a.tobytes() == got[1][1][v].astype(np.float64).tobytes(), (small, large, v)
            if dtype == "f32":
                for (Wg, bg), (Wr, br) in zip(oracle.unpack(a, dims), oracle.unpack(want[v], dims)):
                    assert np.max(np.abs(Wg - Wr)) <= 1e-5 * max(np.max(np.abs(Wr)), 1e-30), (small, v)
                    assert np.max(np.abs(bg - br)) <= 1e-5 * max(np.max(np.abs(br)), 1e-3), (small, v)
            else:
                assert np.linalg.norm(a - want[v]) <= 2.0 ** -7 * np.linalg.norm(want[v] - start), (small, v)

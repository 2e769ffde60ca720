"""A variant's export (canonical parameters and mask, written on the device)
at the edges of its 32 x 32 blocks, bit for bit: the initial state against the
oracle, imported parameters against themselves under the mask, either output
alone, and the state in the middle of an epoch against the epoch's end."""
import ctypes

import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("workload", [1, 3])                    # a full-precision and a bf16 one
@pytest.mark.parametrize("dims", [[37, 33, 5], [64, 32, 32], [33, 65, 31, 2], [96, 256, 10], [40, 7]])
def test_export_is_exact(dims, workload):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2310_10211_amd as g
    P, batch = 3, 16
    cfg = synthetic.config(workload, P=P, dims=dims, batch=batch, lr=(0.05, 0.1), dens=(0.3, 0.9))
    data = synthetic.dataset(cfg, 3 * batch, 40)
    for k in ("x_train", "x_test"):
        data[k] = np.ascontiguousarray(data[k][:, :dims[0]])
    for k in ("y_train", "y_test"):
        data[k] = data[k] % dims[-1]
    print(f"[gpu] export dims={dims} {cfg['dtype']}", flush=True)
    pop = g.Population(cfg, data["x_train"], data["y_train"], data["x_test"], data["y_test"])
    init = oracle.population(cfg, range(P))
    rng = np.random.default_rng(5)
    for v in range(P):
        e = pop.export(v)
        assert np.array_equal(e["mask"], init[v]["mask"])
        assert np.array_equal(e["params"], np.asarray(init[v]["params"], np.float32))
    pop.train_steps(0, 0, 1)
    mid = [pop.export(v)["params"] for v in range(P)]           # in the middle of an epoch
    assert not np.array_equal(mid[0], init[0]["params"])
    pop.train_steps(0, 1, 3)
    p = rng.normal(size=mid[0].size).astype(np.float32)
    pop.import_params(1, p)
    got = pop.export(1)
    off = moff = 0
    for K, N in zip(dims[:-1], dims[1:]):                       # pruned weights are imported as +0
        m = got["mask"][moff:moff + K * N] != 0
        assert np.array_equal(got["params"][off:off + K * N], np.where(m, p[off:off + K * N], np.float32(0)))
        assert np.array_equal(got["params"][off + K * N:off + K * N + N], p[off + K * N:off + K * N + N])
        off += K * N + N
        moff += K * N
    only = np.zeros_like(p)
    assert g.lib().gevo_pop_export(pop._h, 1, g._fp(only), None, None, None) == 0
    assert np.array_equal(only, got["params"])
    mask = np.zeros_like(got["mask"])
    assert g.lib().gevo_pop_export(pop._h, 1, None, mask.ctypes.data_as(ctypes.POINTER(ctypes.c_uint8)), None,
                                   None) == 0
    assert np.array_equal(mask, got["mask"])
    pop.close()

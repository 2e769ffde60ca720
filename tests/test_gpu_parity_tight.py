"""Tighter GPU parity: element-wise single steps of every training kernel,
per-sample prediction, and the argmax tie and NaN-logit rules on the GPU.

* One SGD step from an imported state, weight and bias updates element by
  element against the oracle in bf16 mode (bounds derived in _check_update), on
  each training path and on both sides of the population sizes that divide them:
  nets whose hidden layers train in the streaming kernel (with the backward GEMM
  and the output kernel), including the full 3072-1024-512-10 width, nets whose
  first layer does and whose second trains beside it, the same nets with fewer
  variants on the tile kernels, and the fused two-layer kernel at variants whose
  column blocks are visited in rotated order.  Each case names the kernels that
  have to have run.
* Prediction of single rows (each variant's test loss is then one sample's
  cross-entropy) on the 784-512-256-10 net of the prediction workload, and a
  ragged three-tile test set against the oracle's per-row logits.
* Argmax ties (lowest index wins) and NaN logits (a miss, NaN loss) built by
  importing weights whose logits are the output biases, on the prediction
  path and, with a learning rate of 0, on the training path.
"""
import math

import numpy as np
import pytest

import oracle
import synthetic
from conftest import training_path

pytestmark = pytest.mark.gpu


def _torch():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _pop(cfg, data, **kw):
    _torch()
    import paper_2310_10211_amd as g
    print(f"[gpu] Population {cfg.get('name', '')} P={cfg['P']} dims={cfg['dims']} dtype={cfg['dtype']} "
          f"batch={cfg.get('batch')} n_train={len(data['y_train'])} n_test={len(data['y_test'])}", flush=True)
    return g.Population(cfg, data["x_train"], data["y_train"], data["x_test"], data["y_test"], **kw)


def _data(i, n_train, n_test, dims):
    c = synthetic.config(i)
    d = synthetic.dataset(c, n_train, n_test)
    if dims[0] != d["x_train"].shape[1]:
        for k in ("x_train", "x_test"):
            d[k] = np.ascontiguousarray(d[k][:, :dims[0]])
    return d


def _check_update(dg, dr, what):
    """One step's update (GPU dg, oracle dr), element by element.

    Both sides round the same operands to bf16; the GPU sums them in fp32 in
    its own order, the oracle exactly, so an operand whose two sums straddle a
    bf16 rounding boundary rounds one ulp apart (2^-8 to 2^-7 of it).  Such a
    flip moves one row or column of the update by one term's ulp, so:
      * median relative error over the elements above 1% of the largest
        update <= 2e-4 (a rounding point missing or misplaced on either side
        gives about 1e-3 on most elements; fp32 summation gives about 1e-7);
      * every element within 1e-2 of the largest update (about 2.5 bf16 ulps
        of the largest term)."""
    scale = max(float(np.max(np.abs(dr))), 1e-30)
    diff = np.abs(dg - dr)
    big = np.abs(dr) > 1e-2 * scale
    med = float(np.median(diff[big] / np.abs(dr[big]))) if np.any(big) else 0.0
    info = (what, "max", float(np.max(diff)) / scale, "median rel", med, "elements over 1e-3 of max",
            int(np.sum(diff > 1e-3 * scale)), "of", diff.size)
    assert med <= 2e-4, info
    assert float(np.max(diff)) <= 1e-2 * scale, info


def _compare_step(got, want, before, dims, what):
    """Weights and biases after one step from the same imported state: the
    updates W_after - W_before (see _check_update); the state before the step
    is identical on both sides, so the parameters differ exactly by the
    difference of the updates."""
    for l, ((Wg, bg), (Wr, br), (W0, b0)) in enumerate(zip(oracle.unpack(got, dims), oracle.unpack(want, dims),
                                                          oracle.unpack(before, dims))):
        _check_update(Wg - W0, Wr - W0, f"{what} layer {l + 1} weights")
        _check_update(bg - b0, br - b0, f"{what} layer {l + 1} biases")


def _one_step_case(cfg, data, variants, path, seed=5):
    dims = cfg["dims"]
    pop = _pop(cfg, data)
    ref = oracle.population(cfg, variants)
    rng = np.random.default_rng(seed)
    perm = oracle.permutation(cfg["seed"], 0, len(data["y_train"]))
    before = {}
    for v in variants:
        st = ref[v]
        p = st["params"] + 0.01 * rng.standard_normal(st["params"].shape)
        pop.import_params(v, p.astype(np.float32))            # masked weights are imported as +0
        before[v] = pop.export(v)["params"].astype(np.float64)
    assert training_path(pop, lambda: pop.train_steps(0, 0, 1)) == path
    got = {v: pop.export(v)["params"].astype(np.float64) for v in variants}
    pop.close()
    for v in variants:
        st = ref[v]
        q = before[v].copy()
        oracle.train_steps("bf16", dims, q, st["mask"], st["lr"], data["x_train"], data["y_train"], perm,
                           cfg["batch"], 0, 1)
        _compare_step(got[v], q, before[v], dims, f"variant {v}")


@pytest.mark.parametrize("dims,batch,n_train,P,path", [
    ([1024, 256, 128, 10], 256, 700, 33, "streamed 2"),     # both hidden layers streamed, batch tile 256
    ([1024, 256, 128, 10], 256, 700, 32, "tiles"),
    ([512, 128, 256, 10], 128, 300, 33, "streamed 2"),      # batch tile 128
    ([512, 128, 256, 10], 128, 300, 3, "tiles"),
    ([512, 128, 10], 250, 300, 65, "streamed 1"),           # one hidden layer, no backward GEMM
    ([3072, 1024, 512, 10], 256, 512, 9, "streamed 2"),     # the full width of the 128-variant CIFAR-shaped workload
    ([3072, 1024, 512, 10], 256, 512, 2, "tiles"),
    ([1024, 256, 160, 10], 256, 300, 65, "streamed 1"),     # the first layer streamed, the second beside it
    ([1024, 256, 160, 10], 256, 300, 64, "tiles"),
    ([512, 384, 70, 10], 128, 300, 43, "streamed 1"),       # a ragged second layer, batch tile 128
    ([512, 1024, 96, 10], 120, 300, 17, "streamed 1"),      # its inputs in two LDS blocks
    ([512, 256, 192, 10], 128, 300, 65, "tiles"),           # less than three quarters of the weights in the first
])
def test_streamed_net_one_step_elementwise(dims, batch, n_train, P, path):
    cfg = synthetic.config(5, P=P, dims=dims, batch=batch, lr=(0.05, 0.05))
    data = _data(5, n_train, 256, dims)
    _one_step_case(cfg, data, sorted({0, 1, P - 1}), path)


# The 784-256-10 bf16 nets with a 128-row batch train in the streaming fused
# kernel from 33 variants up and on the tile kernels below; GEVO_RESIDENT=1
# selects the resident kernel (a pair of workgroups per variant) for the same
# shapes.
KERNELS = ["resident", "streaming"]
RUNS = [("resident", 24, "fused"), ("streaming", 24, "tiles"), ("streaming", 40, "fused")]


def _select_kernel(monkeypatch, kernel):
    if kernel == "resident":
        monkeypatch.setenv("GEVO_RESIDENT", "1")
    else:
        monkeypatch.delenv("GEVO_RESIDENT", raising=False)


@pytest.mark.parametrize("kernel,P,path", RUNS)
def test_fused_kernel_rotated_block_order_one_step_elementwise(kernel, P, path, monkeypatch):
    """Variant v of the streaming fused kernel visits its column blocks from
    block (v / 8) mod 25: variants 8, 23 and 39 start at blocks 1, 2 and 4.  In the
    resident kernel variants 16 and 23 are the second pairs of their XCDs."""
    _select_kernel(monkeypatch, kernel)
    cfg = synthetic.config(3, P=P, lr=(0.05, 0.2))
    data = _data(3, 256, 256, cfg["dims"])
    _one_step_case(cfg, data, [0, 8, 16, 23] + ([39] if P > 24 else []), path)


@pytest.mark.parametrize("kernel,P,path", RUNS)
def test_fused_kernel_rotated_block_order_epoch(kernel, P, path, monkeypatch):
    _select_kernel(monkeypatch, kernel)
    cfg = synthetic.config(3, P=P)
    data = _data(3, 700, 300, cfg["dims"])
    pop = _pop(cfg, data)
    assert training_path(pop, lambda: pop.train_epoch(0)) == path
    pop.predict()
    s = pop.scores()
    pop.close()
    ref = oracle.evaluate(cfg, data, variants=[9, 17, 23], epochs=1)
    for v in (9, 17, 23):
        r = ref[v]
        assert abs(float(s["train_loss"][v]) - r["train_loss"][-1]) <= 2e-2 * abs(r["train_loss"][-1]), v
        assert abs(float(s["test_loss"][v]) - r["test_loss"]) <= 2e-2 * abs(r["test_loss"]), v
        assert abs(float(s["train_acc"][v]) - r["train_acc"][-1]) <= 0.005, v


@pytest.mark.parametrize("P,path", [(20, "tiles"), (36, "fused")])
def test_resident_and_streaming_fused_kernels_agree(P, path, monkeypatch):
    """The resident kernel and the one that the population otherwise trains in,
    on one population (a ragged last batch of 20 rows, more variants than one
    dispatch round of pairs would need on a small grid): per-variant scores and
    the trained weights agree to the bf16 rounding of their different fp32
    summation orders."""
    cfg = synthetic.config(3, P=P)
    data = _data(3, 1300, 300, cfg["dims"])
    out = {}
    for kernel in KERNELS:
        _select_kernel(monkeypatch, kernel)
        pop = _pop(cfg, data)
        assert training_path(pop, lambda: pop.train_epoch(0)) == ("fused" if kernel == "resident" else path)
        pop.predict()
        out[kernel] = (pop.scores(), [pop.export(v)["params"] for v in range(cfg["P"])])
        pop.close()
    (sa, pa), (sb, pb) = out["resident"], out["streaming"]
    for k in ("train_loss", "test_loss"):
        assert np.allclose(sa[k], sb[k], rtol=1e-2, atol=0), k
    for k in ("train_acc", "test_acc"):
        assert np.max(np.abs(sa[k] - sb[k])) <= 0.01, k
    for v in range(cfg["P"]):
        a, b = pa[v].astype(np.float64), pb[v].astype(np.float64)
        assert np.array_equal(a == 0, b == 0), v           # masked weights +0 in both
        big = np.abs(b) > 1e-2 * np.max(np.abs(b))
        rel = np.abs(a[big] - b[big]) / np.abs(b[big])
        assert np.median(rel) <= 1e-3 and np.max(np.abs(a - b)) <= 2e-2 * np.max(np.abs(b)), v


# --------------------------------------------------------------- prediction
def _predict_cfg(P, dims=(784, 512, 256, 10)):
    return synthetic.config(4, P=P, dims=list(dims))


def test_prediction_single_rows_per_sample_ce():
    """With one test row, each variant's test loss is that row's
    cross-entropy and its accuracy that row's hit (prediction workload net,
    each variant a noisy, pruned copy of the base)."""
    cfg = _predict_cfg(16)
    full = _data(4, 0, 40, cfg["dims"])
    ref = oracle.population(cfg)
    for i in (0, 13, 37):
        data = dict(x_train=full["x_train"], y_train=full["y_train"], x_test=full["x_test"][i:i + 1].copy(),
                    y_test=full["y_test"][i:i + 1].copy())
        pop = _pop(cfg, data)
        pop.predict()
        s = pop.scores()
        pop.close()
        for v in range(cfg["P"]):
            ce, _, logits, _ = oracle.batch_grad("bf16", cfg["dims"], ref[v]["params"], data["x_test"], data["y_test"])
            assert abs(float(s["test_loss"][v]) - ce) <= 2e-3 * abs(ce) + 1e-5, (i, v, s["test_loss"][v], ce)
            z = logits[0]
            top = np.sort(z)[::-1]
            if top[0] - top[1] > 1e-2 * max(1.0, abs(top[0])):
                hit = float(int(np.argmax(z)) == int(data["y_test"][0]))
                assert float(s["test_acc"][v]) == hit, (i, v)


def test_prediction_ragged_tiles_against_oracle_logits():
    """Three 256-row tiles with a ragged tail of 88 rows: mean loss per
    variant against the oracle's per-row losses within 1e-3, and hits equal
    except on rows whose top two oracle logits are within 1e-2."""
    cfg = _predict_cfg(8)
    data = _data(4, 0, 600, cfg["dims"])
    pop = _pop(cfg, data)
    pop.predict()
    s = pop.scores()
    pop.close()
    ref = oracle.population(cfg)
    n = len(data["y_test"])
    for v in range(cfg["P"]):
        ce, _, logits, _ = oracle.batch_grad("bf16", cfg["dims"], ref[v]["params"], data["x_test"], data["y_test"])
        assert abs(float(s["test_loss"][v]) - ce / n) <= 1e-3 * abs(ce / n), (v, s["test_loss"][v], ce / n)
        top2 = np.sort(logits, axis=1)[:, ::-1]
        close = int(np.sum(top2[:, 0] - top2[:, 1] <= 1e-2 * np.maximum(1.0, np.abs(top2[:, 0]))))
        hits = int(np.sum(np.argmax(logits, axis=1) == data["y_test"]))
        assert abs(round(float(s["test_acc"][v]) * n) - hits) <= close, (v, s["test_acc"][v] * n, hits, close)


# ------------------------------------------------- ties and NaN logits
C = 10
_BIASES = [
    np.zeros(C),                                                        # ten-way tie: class 0
    np.array([0, 0, 0, 1, 0, 0, 0, 1, 0, 0], float),                    # tie of 3 and 7: class 3
    np.array([0, 0, 0, 0, 0, np.nan, 0, 0, 0, 0], float),               # a NaN logit: a miss, NaN loss
    np.array([0, 0, 0, 0, 0, 0, 0, 0, 0, 1], float),                    # class 9
]
_PRED = [0, 3, None, 9]


def _expected(bias, y):
    """Closed forms for logits equal to `bias` on every row: accuracy and
    mean cross-entropy log(sum exp b) - b_y."""
    if np.any(np.isnan(bias)):
        return 0.0, math.nan
    lse = math.log(float(np.sum(np.exp(bias))))
    pred = int(np.argmax(bias))                                         # numpy: lowest index on ties
    return float(np.mean(y == pred)), float(np.mean(lse - bias[y]))


def _tie_params(dims, v_bias):
    """Hidden layers: small random weights; output layer weights 0
    and biases v_bias, so the logits equal v_bias on every row."""
    rng = np.random.default_rng(11)
    parts = []
    for l in range(1, len(dims)):
        din, dout = dims[l - 1], dims[l]
        if l < len(dims) - 1:
            parts += [0.05 * rng.standard_normal(din * dout), np.zeros(dout)]
        else:
            parts += [np.zeros(din * dout), v_bias]
    return np.concatenate(parts).astype(np.float32)


@pytest.mark.parametrize("i,dims", [
    (3, [784, 256, 10]),            # bf16: prediction GEMM with the output layer fused
    (5, [1024, 256, 128, 10]),      # bf16, three layers
    (2, [784, 96, 10]),             # fp32
    (1, [256, 10]),                 # fp32, output layer only (784 fp32 inputs exceed its LDS tile)
])
def test_prediction_argmax_ties_and_nan_logits(i, dims):
    cfg = synthetic.config(i, P=4, dims=dims, dens=(1.0, 1.0), dens_list=None)
    cfg.pop("dens_list", None)
    data = _data(i, 0, 300, dims)
    pop = _pop(cfg, data)
    for v, b in enumerate(_BIASES):
        pop.import_params(v, _tie_params(dims, b))
    pop.predict()
    s = pop.scores()
    pop.close()
    for v, b in enumerate(_BIASES):
        acc, ce = _expected(b, data["y_test"])
        assert float(s["test_acc"][v]) == pytest.approx(acc, abs=1e-7), (v, s["test_acc"][v], acc)
        if math.isnan(ce):
            assert math.isnan(float(s["test_loss"][v])), v
        else:
            assert float(s["test_loss"][v]) == pytest.approx(ce, rel=1e-5), (v, s["test_loss"][v], ce)


@pytest.mark.parametrize("i,dims,batch,P,path", [
    (3, [784, 256, 10], 128, 33, "fused"),
    (3, [784, 256, 10], 128, 4, "tiles"),
    (3, [784, 256, 10], 64, 4, "fused"),                    # batch tile 64
    (5, [1024, 256, 128, 10], 256, 33, "streamed 2"),       # streaming, backward GEMM and output kernels
    (5, [1024, 256, 128, 10], 256, 4, "tiles"),
    (2, [784, 96, 10], 64, 4, "tiles"),                     # fp32
])
def test_training_argmax_ties_and_nan_logits(i, dims, batch, P, path):
    """Learning rate 0: the training-split accuracy and loss of an epoch are
    the same closed forms over the training labels; a NaN logit leaves its
    variant at accuracy 0 and NaN loss and the other variants untouched."""
    cfg = synthetic.config(i, P=P, dims=dims, batch=batch, lr=(0.0, 0.0), dens=(1.0, 1.0))
    cfg.pop("dens_list", None)
    data = _data(i, 500, 256, dims)
    pop = _pop(cfg, data)
    for v, b in enumerate(_BIASES):
        pop.import_params(v, _tie_params(dims, b))
    assert training_path(pop, lambda: pop.train_epoch(0)) == path
    s = pop.scores()
    pop.close()
    for v, b in enumerate(_BIASES):
        acc, ce = _expected(b, data["y_train"])
        assert float(s["train_acc"][v]) == pytest.approx(acc, abs=1e-7), (v, s["train_acc"][v], acc)
        if math.isnan(ce):
            assert math.isnan(float(s["train_loss"][v])), v
        else:
            assert float(s["train_loss"][v]) == pytest.approx(ce, rel=1e-5), (v, s["train_loss"][v], ce)

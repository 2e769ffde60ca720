"""Convolutional prediction in whole segments at the edges of its tiles,
against the oracle and against the layer-by-layer kernels (which a prediction
with kernel-level timing runs): rows of at most 8, 16 and 32 pixels, full and
ragged, both strides on each, 32 to 256 contracted channels, one to several
segments, one to several images per group and groups per workgroup, a ragged
last group and launch, and every pooling run."""
import numpy as np
import pytest

import synthetic
from oracle import cnn

pytestmark = pytest.mark.gpu

# H, W, C, stem, blocks, n_test, P
SHAPES = [
    (32, 32, 3, 32, [(1, 128), (2, 128), (1, 256)], 9, 2),       # 32-wide rows, both strides; pooled map of 256
    (24, 24, 1, 64, [(2, 256), (1, 128)], 7, 2),                 # ragged 32- and 16-wide rows
    (12, 20, 2, 32, [(2, 128)], 5, 3),                           # not square; odd channel count of a window row
    (16, 16, 4, 128, [(1, 128), (1, 128), (2, 256), (1, 128)], 6, 2),   # two segments; 16-wide rows
    (16, 16, 3, 32, [(2, 256), (2, 128)], 11, 3),                # 256 contracted channels, 8-wide rows, stride 2
    (8, 8, 3, 256, [(1, 256), (1, 256), (2, 128)], 13, 2),       # 8-wide rows, 256 contracted channels twice
    (8, 10, 3, 32, [(2, 128), (1, 128)], 10, 3),                 # rows of 10 and of 5; pooled map of 20
    (12, 12, 3, 32, [(1, 128)], 9, 3),                           # pooled map of 144
    (8, 4, 3, 32, [(2, 128)], 21, 3),                            # pooled map of 8
    (4, 4, 1, 32, [(1, 128)], 19, 3),                            # pooled map of 16, narrow rows
    (7, 7, 3, 32, [(2, 128)], 11, 3),                            # odd images back to back: an odd element count each
    (15, 15, 1, 64, [(2, 128), (1, 128)], 19, 3),
    (31, 31, 3, 32, [(2, 128), (2, 128)], 6, 2),
    (4, 4, 3, 32, [(2, 128), (1, 128)], 4170, 9),                # pooled map of 4; two launches, two groups a workgroup
]


@pytest.mark.parametrize("H,W,C,stem,blocks,n_test,P", SHAPES)
def test_segments_match_the_oracle_and_the_layers(H, W, C, stem, blocks, n_test, P):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2310_10211_amd as g
    cfg = synthetic.cnn_config("small", name="segments", P=P, H=H, W=W, C=C, stem=stem, blocks=blocks, classes=10,
                               n_test=n_test, seed=91)
    base, x, y = synthetic.cnn_inputs(cfg)
    print(f"[gpu] segments {H}x{W}x{C} stem={stem} blocks={blocks} n_test={n_test} P={P}", flush=True)
    pop = g.CnnPopulation(cfg, base, x, y)
    pop.predict()
    s = pop.scores()
    pop.predict()                                                # the same again
    assert np.array_equal(pop.scores()["test_loss"], s["test_loss"])
    pop.set_profiling(True)
    pop.predict()
    layers = pop.scores()
    pop.set_profiling(False)
    # Bar as for the layer-by-layer kernels against the oracle: the same
    # values are rounded to bf16, the sums in fp32 differ in order, so single
    # activations move by one bf16 ulp (2^-8) with probability about K 2^-16
    # and the mean loss by far less than 2e-3.
    for v in range(P):
        assert abs(s["test_loss"][v] - layers["test_loss"][v]) <= 2e-3 * abs(layers["test_loss"][v]), v
        assert abs(s["test_acc"][v] - layers["test_acc"][v]) * n_test <= max(1, n_test // 200) + 1e-3, v
    sample = sorted({0, P - 1})
    ref = cnn.evaluate(cfg, base.astype(np.float64), x, y, sample, mode="bf16")
    for v in sample:
        ce, corr = ref[v]
        assert abs(s["test_loss"][v] - ce / n_test) <= 2e-3 * abs(ce / n_test), v
        assert abs(round(float(s["test_acc"][v]) * n_test) - corr) <= max(1, n_test // 200), v
    # a removed layer reaches the segment kernel's weights
    before = s["test_loss"][P - 1]
    pop.remove_layer(P - 1, "pw0")
    pop.predict()
    a = pop.scores()["test_loss"]
    assert a[P - 1] != before and np.array_equal(a[:P - 1], s["test_loss"][:P - 1])
    pop.set_profiling(True)
    pop.predict()
    b = pop.scores()["test_loss"]
    assert abs(a[P - 1] - b[P - 1]) <= 2e-3 * abs(b[P - 1])
    pop.close()

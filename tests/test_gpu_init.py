"""Population init at the edges of its two kernels (four inputs of a unit to a
thread where their number is a multiple of four, a unit's 32 inputs else):
masks and weights of plain, noisy and genome populations against the oracle,
with one and several variants to a thread."""
import numpy as np
import pytest

import oracle
import synthetic
from oracle import nsga2 as ns

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,P", [([36, 40, 20, 5], 3), ([4, 33, 2], 3), ([100, 30, 32], 700), ([784, 128, 10], 50),
                                    ([37, 40, 22, 5], 3), ([6, 64, 3], 70)])
def test_init_and_genomes_are_the_oracles(dims, P):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2310_10211_amd as g
    print(f"[gpu] init dims={dims} P={P}", flush=True)
    sample = sorted({0, 1, 2, P // 2, P - 1})
    x, y = np.zeros((8, dims[0]), np.float32), np.zeros(8, np.int32)
    for over in (dict(init="xavier"), dict(init="base_noise", noise_std=0.05)):
        cfg = synthetic.config(3, P=P, dims=dims, batch=8, dens=(0.3, 0.9), **over)
        pop = g.Population(cfg, x, y, x, y)
        ref = oracle.population(cfg, sample)
        for v in sample:
            e = pop.export(v)
            assert np.array_equal(e["mask"], ref[v]["mask"]), v
            if over["init"] == "xavier":
                assert np.array_equal(e["params"], np.asarray(ref[v]["params"], np.float32)), v
            else:                              # the noise's normal deviate is a binary32 log and cos here, fp64 there
                np.testing.assert_allclose(e["params"], ref[v]["params"], rtol=2e-6, atol=0)
        pop.close()
    cfg = synthetic.config(3, P=P, dims=dims, batch=8, dens=(0.3, 0.9))
    pop = g.Population(cfg, x, y, x, y)
    genomes = [ns.initial(1, 100 + v, 0.3, id_base=10 * v)[0] if v % 7 else [] for v in range(P)]
    width = max(1, dims[1] - 3)
    genomes[1] = genomes[1] + [(g.EDIT_WIDTH, 1, width), (g.EDIT_BIAS_OFF, 1, 0)]
    pop.set_genomes(genomes, 0.05)
    full, _ = oracle.variant_init(cfg["seed"], 0, dims, 1 << 24)
    for v in sample:
        plain = [e for e in genomes[v] if e[0] not in (g.EDIT_WIDTH, g.EDIT_BIAS_OFF)]
        _, ids, th, _ = ns.apply(plain, 0.05)
        mask = oracle.genome_mask(cfg["seed"], dims, ids, th)
        off = moff = 0
        want, e = full.copy(), pop.export(v)
        for l, (K, N) in enumerate(zip(dims[:-1], dims[1:])):
            m = mask[moff:moff + K * N].reshape(K, N).copy()
            if v == 1 and l == 0:
                m[:, width:] = 0
            if v == 1 and l == 1:
                m[width:] = 0
            assert np.array_equal(e["mask"][moff:moff + K * N], m.reshape(-1)), (v, l)
            want[off:off + K * N] *= m.reshape(-1)
            off += K * N + N
            moff += K * N
        assert np.array_equal(e["params"].astype(np.float64), want), v
    pop.close()

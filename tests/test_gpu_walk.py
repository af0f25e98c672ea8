"""The data-driven kernels against the generated ones, bit for bit: few rows of
a specialised model (gathered) equal the same rows in a large call (generated
kernel), and a generic model's histograms equal the specialised model's."""
import numpy as np
import pytest

from paper_2511_09376_amd import synth
from tests.gpu_util import assert_phi_close
from tests.test_gpu_parity import _edge_ensemble

torch = pytest.importorskip("torch")
import oracle  # noqa: E402

pytestmark = pytest.mark.gpu

# edge: root leaf, stump, repeats, depth-8 chain; pool: 1600 units on 3 of 8
# features (several chunks of units); deep: 200 features (row keys not staged),
# 512-entry quads (16-bit slots)
ENSEMBLES = {
    "edge": _edge_ensemble,
    "pool": lambda: synth.make_ensemble(synth.ModelSpec(200, 4, 4, 0.0, 8, feature_pool=3),
                                        synth.DataSpec(8, False, 0.05), 11),
    "deep": lambda: synth.make_ensemble(synth.ModelSpec(6, 8, 8, 0.0, 200), synth.DataSpec(200, True, 0.05), 3),
}


@pytest.fixture(scope="module", params=sorted(ENSEMBLES))
def loaded(request):
    from paper_2511_09376_amd import wdf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ens = ENSEMBLES[request.param]()
    ctx = wdf.Context(0)
    F, n = ens.n_features, 5000
    rng = np.random.default_rng(7)
    X = rng.normal(size=(F, n)).astype(np.float32)
    X[rng.random((F, n)) < 0.05] = np.nan
    inner = ens.feature >= 0
    f, t = ens.feature[inner], ens.threshold[inner]
    for c, vals in enumerate((t, -np.inf, np.inf, np.nan, 0.0, -0.0)):   # on thresholds, and the special values
        X[f, c] = vals
    return wdf, ens, ctx, torch.from_numpy(X).cuda(), X


def test_few_rows_equal_many(loaded):
    wdf, ens, ctx, X, _ = loaded
    model = wdf.Model(ctx, ens)
    assert model.specialised
    for kind in (wdf.SHAPLEY, wdf.BANZHAF):
        bg = wdf.Background(model, X[:, :777].contiguous(), values=kind)
        ref = bg.explain(X)                                # 5000 rows: the generated kernel
        for n in (1, 2, 4, 5, 16, 17, 63, 64, 65, 512, 1025, 2047, 2048, 2049):
            for a in (0, 3):                               # a slice: ldx > n, rows not 16-byte aligned
                assert torch.equal(bg.explain(X[:, a:a + n]), ref[:, a:a + n]), f"n={n} from {a}"
        wide = torch.full((ens.n_features, 100), 7.0, device="cuda")
        bg.explain(X[:, :33], out=wide[:, 10:43])          # ldphi > n: nothing else written
        assert torch.equal(wide[:, 10:43], ref[:, :33])
        assert bool((wide[:, :10] == 7).all()) and bool((wide[:, 43:] == 7).all())


def test_generic_histograms_and_phi(loaded):
    wdf, ens, ctx, X, Xn = loaded
    spec, gen = wdf.Model(ctx, ens), wdf.Model(ctx, ens, wdf.KERNEL_GENERIC)
    for m in (1, 63, 64, 65, 777, 5000):
        a, b = wdf.Background(spec, X[:, :m]), wdf.Background(gen, X[:, :m])
        np.testing.assert_array_equal(a.histograms(), b.histograms())
        np.testing.assert_array_equal(a.tables(), b.tables())
    b = wdf.Background(gen, X[:, :300])
    phi = b.explain(X)
    assert torch.equal(b.explain(X[:, 11:111]), phi[:, 11:111])
    ref = oracle.bg_walk(oracle.Model(ens), np.ascontiguousarray(Xn[:, :40]), np.ascontiguousarray(Xn[:, :300]))
    assert_phi_close(phi[:, :40].cpu().numpy(), ref)


@pytest.mark.parametrize("name,rows,many", [("trees", (1, 3, 64, 65, 512, 513, 1025), 8192),   # many: the generated kernels
                                            ("pool", (1, 5, 64, 130, 512), 4000)])             # many: the generic ones
def test_few_interaction_rows_equal_many(name, rows, many):
    from paper_2511_09376_amd import wdf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    data = synth.DataSpec(127 if name == "trees" else 8, False, 0.05)
    ens = ENSEMBLES["pool"]() if name == "pool" else synth.make_ensemble(synth.ModelSpec(20, 6, 6, 0.0, 127), data, 5)
    X = torch.from_numpy(synth.make_matrix(data, many, 9)).cuda()
    bg = wdf.Background(wdf.Model(wdf.Context(0), ens), X[:, :999].contiguous(), values=wdf.SHAPLEY_IV)
    ref = bg.explain_iv(X)
    for n in rows:
        assert torch.equal(bg.explain_iv(X[:, 7:7 + n]), ref[:, :, 7:7 + n]), f"n={n}"

"""The data-driven gather bit for bit against the generated explain kernel and
against the oracle, on models that take it (asserted): irregular trees (root
leaf, stump, repeats, single leaves, a depth-8 chain, 16-bit slots) and columns
whose units span several chunks.  Few-feature models keep the generated kernel."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2511_09376_amd import synth
from tests.gpu_util import assert_phi_close
from tests.test_gpu_parity import _edge_ensemble

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wdf():
    from paper_2511_09376_amd import wdf as w
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return w


@pytest.fixture(scope="module")
def ctx(wdf):
    return wdf.Context(0)


def _irregular():
    a = _edge_ensemble()
    b = synth.make_ensemble(synth.ModelSpec(60, 1, 8, 0.2, 40), synth.DataSpec(40, False, 0.05), 21)
    cat = {f.name: np.concatenate([getattr(a, f.name), getattr(b, f.name)]) for f in dataclasses.fields(a)
           if f.name not in ("n_features", "node_offset")}
    return dataclasses.replace(b, node_offset=np.r_[a.node_offset, b.node_offset[1:] + a.node_offset[-1]], **cat)


def _chunks():   # 1600 units, of which a block of 4 columns needs nearly all: 512 at a time
    return synth.make_ensemble(synth.ModelSpec(100, 6, 6, 0.0, 8), synth.DataSpec(8, False, 0.05), 11)


def _rows(ens, n):
    rng = np.random.default_rng(7)
    X = rng.normal(size=(ens.n_features, n)).astype(np.float32)
    X[rng.random(X.shape) < 0.05] = np.nan
    inner = ens.feature >= 0
    for c, v in enumerate((ens.threshold[inner], -np.inf, np.inf, np.nan, 0.0, -0.0)):
        X[ens.feature[inner], c] = v
    return X


@pytest.mark.parametrize("make", [_irregular, _chunks])
@pytest.mark.parametrize("pairs", [False, True], ids=["quads", "pairs"])
def test_gather_equals_the_generated_kernel(wdf, ctx, make, pairs):
    ens = make()
    Xn = _rows(ens, 3000)
    X = torch.from_numpy(Xn).cuda()
    model = wdf.Model(ctx, ens, wdf.KERNEL_SPECIALISED | (wdf.KERNEL_PAIRS if pairs else 0))
    for kind in (wdf.SHAPLEY, wdf.BANZHAF):
        bg = wdf.Background(model, X[:, :777].contiguous(), values=kind)
        assert bg.explain_route(3000) == wdf.ROUTE_GENERATED
        ref = bg.explain(X)
        for n in (1, 2, 5, 17, 63, 64, 65, 513, 1025, 2048):
            assert bg.explain_route(n) == wdf.ROUTE_GATHER
            for a in (0, 3):
                assert torch.equal(bg.explain(X[:, a:a + n]), ref[:, a:a + n]), f"n={n} from {a}"
    bg = wdf.Background(model, X[:, :300].contiguous())
    got = bg.explain(X[:, :24].contiguous()).cpu().numpy()
    assert_phi_close(got, oracle.bg_walk(oracle.Model(ens), np.ascontiguousarray(Xn[:, :24]),
                                         np.ascontiguousarray(Xn[:, :300]), threads=8))


@pytest.mark.parametrize("spec", [(200, 4, 8, 3), (400, 4, 4, 4), (40, 6, 8, 8)])
def test_few_features_keep_the_generated_kernel(wdf, ctx, spec):
    """One feature takes a value from more than half of the units, and the
    tables fit the L2."""
    trees, depth, F, pool = spec
    ens = synth.make_ensemble(synth.ModelSpec(trees, depth, depth, 0.0, F, feature_pool=pool),
                              synth.DataSpec(F, False, 0.05), 11)
    X = torch.from_numpy(_rows(ens, 600)).cuda()
    model, generic = wdf.Model(ctx, ens, wdf.KERNEL_SPECIALISED), wdf.Model(ctx, ens, wdf.KERNEL_GENERIC)
    a, b = wdf.Background(model, X[:, :99].contiguous()), wdf.Background(generic, X[:, :99].contiguous())
    for n in (1, 64, 600):
        assert a.explain_route(n) == wdf.ROUTE_GENERATED and b.explain_route(n) == wdf.ROUTE_GATHER
        torch.testing.assert_close(a.explain(X[:, :n]), b.explain(X[:, :n]), rtol=0, atol=1e-5 * float(b.explain(X).abs().max()))


# trees, depths, features: stumps; unused features; 80 units in chunks of 64; a unit
# of 512 entries (16-bit slots); a chunk of exactly 64
@pytest.mark.parametrize("spec", [(3, 1, 1, 4), (2, 2, 2, 60), (40, 3, 3, 160), (1, 8, 8, 30), (30, 1, 8, 300), (16, 4, 4, 20)])
def test_small_generic_models_with_many_rows(wdf, ctx, spec):
    """Blocks of 512 rows (at least 2048 rows per unit of a chunk) against blocks
    of few rows, bit for bit, and the oracle; nothing outside the output."""
    trees, lo, hi, F = spec
    ens = synth.make_ensemble(synth.ModelSpec(trees, lo, hi, 0.1 if lo != hi else 0.0, F), synth.DataSpec(F, False, 0.05), 5)
    n = 2048 * 64 + 333
    head = _rows(ens, 4000)
    X = torch.from_numpy(head).cuda().repeat(1, n // 4000 + 1)[:, :n + 1]
    model = wdf.Model(ctx, ens, wdf.KERNEL_GENERIC)
    bg = wdf.Background(model, X[:, :500].contiguous())
    few = bg.explain(X[:, :1024])
    out = torch.full((F, n + 70), 7.0, device="cuda")
    bg.explain(X[:, :n], out=out[:, 33:33 + n])                      # a slice: strides, ragged last block
    assert bool((out[:, :33] == 7).all()) and bool((out[:, 33 + n:] == 7).all())
    phi = out[:, 33:33 + n]
    assert torch.equal(phi[:, :1024], few)
    for a in (1024, 4000 * 7 + 5, n - 1024):
        assert torch.equal(phi[:, a:a + 1024], bg.explain(X[:, a:a + 1024])), a
    ref = oracle.bg_walk(oracle.Model(ens), np.ascontiguousarray(head[:, :24]), np.ascontiguousarray(head[:, :500]), threads=8)
    assert_phi_close(phi[:, :24].cpu().numpy(), ref)


@pytest.mark.parametrize("spec", [(3, 2, 4), (2, 2, 60)])
def test_small_interaction_models_with_many_rows(wdf, ctx, spec):
    trees, depth, F = spec
    ens = synth.make_ensemble(synth.ModelSpec(trees, depth, depth, 0.0, F), synth.DataSpec(F, False, 0.05), 5)
    n = 40_001
    X = torch.from_numpy(_rows(ens, n)).cuda()
    bg = wdf.Background(wdf.Model(ctx, ens, wdf.KERNEL_GENERIC), X[:, :500].contiguous(), values=wdf.BANZHAF_IV)
    assert bg.explain_route(n) == wdf.ROUTE_GATHER
    iv = bg.explain_iv(X)
    for a in (0, 20_003, n - 700):
        assert torch.equal(iv[:, :, a:a + 700], bg.explain_iv(X[:, a:a + 700])), a
    ref = oracle.bg_iv_walk(oracle.Model(ens), np.ascontiguousarray(X[:, :16].cpu().numpy()),
                            np.ascontiguousarray(X[:, :500].cpu().numpy()), oracle.BANZHAF, threads=8)
    g = iv[:, :, :16].cpu().numpy().reshape(F * F, -1)
    assert (np.abs(g - ref.reshape(F * F, -1)).max(0) / np.maximum(np.abs(ref).reshape(F * F, -1).max(0), 1e-30)).max() <= 1e-5

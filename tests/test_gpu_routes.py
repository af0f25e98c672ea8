"""Which kernels an explain call runs (wdf_debug_explain_route), by its buffers
(phi over X, interaction values over X, column slices of one matrix) and by the
model and the rows, and that the values do not depend on it."""
import numpy as np
import pytest

import oracle
from paper_2511_09376_amd import synth

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


@pytest.fixture(scope="module")
def trees(wdf, ctx):
    """30 depth-5 trees of 30 features (6 explain stages), and 6000 rows."""
    data = synth.DataSpec(30, False, 0.05)
    ens = synth.make_ensemble(synth.ModelSpec(30, 5, 5, 0.0, 30), data, 5)
    return wdf.Model(ctx, ens, wdf.KERNEL_SPECIALISED), torch.from_numpy(synth.make_matrix(data, 6000, 9)).cuda()


@pytest.mark.parametrize("n", [1, 65, 1000, 2048, 2049, 5000])
def test_explain_in_place(wdf, trees, n):
    model, X = trees
    bg = wdf.Background(model, X[:, :500].contiguous())
    ref = bg.explain(X[:, 17:17 + n])
    assert bg.explain_route(n) == (wdf.ROUTE_GATHER if n <= 2048 else wdf.ROUTE_GENERATED)
    Y = X[:, 17:17 + n].contiguous()
    assert bg.explain_route(n, Y, Y) == wdf.ROUTE_GENERATED
    bg.explain(Y, out=Y)
    assert torch.equal(Y, ref)
    W = X.clone()
    Y = W[:, 17:17 + n]                      # a column slice, the rows around it kept
    bg.explain(Y, out=Y)
    assert torch.equal(W[:, 17:17 + n], ref)
    assert torch.equal(W[:, :17].view(torch.int32), X[:, :17].view(torch.int32))
    assert torch.equal(W[:, 17 + n:].view(torch.int32), X[:, 17 + n:].view(torch.int32))


def test_slices_of_one_matrix_share_nothing(wdf, trees):
    model, X = trees
    bg = wdf.Background(model, X[:, :500].contiguous())
    W = X.clone()
    for a, b, n, shared in ((0, 100, 100, False), (100, 0, 100, False), (5, 104, 100, True), (104, 5, 100, True),
                            (0, 5900, 100, False), (5900, 0, 100, False)):
        Y, out = W[:, a:a + n], W[:, b:b + n]
        assert bg.explain_route(n, Y, out) == (wdf.ROUTE_GENERATED if shared else wdf.ROUTE_GATHER), (a, b)
    assert bg.explain_route(100, W[:, :100], W[:, :200][:, 50:150]) == wdf.ROUTE_GENERATED
    ref = bg.explain(X[:, :100])
    bg.explain(W[:, :100], out=W[:, 100:200])
    assert torch.equal(W[:, 100:200], ref)


@pytest.mark.parametrize("kname", ["specialised", "generic"])
def test_interaction_values_over_their_rows(wdf, ctx, trees, kname):
    """X inside the output: every pattern is taken before a value is stored."""
    model, X = trees
    if kname == "generic":
        ens = synth.make_ensemble(synth.ModelSpec(30, 5, 5, 0.0, 30), synth.DataSpec(30, False, 0.05), 5)
        model = wdf.Model(ctx, ens, wdf.KERNEL_GENERIC)
    bg = wdf.Background(model, X[:, :500].contiguous(), values=wdf.SHAPLEY_IV)
    for n in (1, 100, 512, 4000):
        ref = bg.explain_iv(X[:, :n])
        out = torch.full((30, 30, n), 7.0, device="cuda")
        Y = out.view(900, n)[435:465]
        Y.copy_(X[:, :n])
        assert bg.explain_route(n, Y, out) != wdf.ROUTE_GATHER
        bg.explain_iv(Y, out=out)
        assert torch.equal(out, ref), n


def test_more_rows_than_one_launch_holds(wdf, ctx):
    """A generic model of one feature: 512 threads per 64 rows pass 2^32 threads
    at 536 870 848 rows."""
    n = 536_870_848 + 1000
    ens = synth.make_ensemble(synth.ModelSpec(1, 2, 2, 0.0, 1), synth.DataSpec(1, False, 0.0), 3)
    model = wdf.Model(ctx, ens, wdf.KERNEL_GENERIC)
    row = torch.linspace(-3, 3, 4099, device="cuda")
    X = row.repeat(n // 4099 + 1)[None, :n]
    bg = wdf.Background(model, X[:, :300].contiguous())
    phi = bg.explain(X)
    assert torch.equal(phi[:, -5000:], bg.explain(X[:, -5000:]))
    assert torch.equal(phi[:, :4099 * 1000].view(1000, 4099), phi[:, :4099].expand(1000, 4099))
    iv = wdf.Background(model, X[:, :300].contiguous(), values=wdf.SHAPLEY_IV)
    assert iv.explain_route(n) == wdf.ROUTE_GATHER            # one feature: no pairs
    phi.fill_(7.0)
    iv.explain_iv(X, out=phi[None])
    assert not phi[:, -5000:].any() and not phi[:, :5000].any() and int(torch.count_nonzero(phi[:, ::4096])) == 0


def _model(trees, depth, F, pool=0):
    data = synth.DataSpec(F, F > 100, 0.05)
    return synth.make_ensemble(synth.ModelSpec(trees, depth, depth, 0.0, F, **({"feature_pool": pool} if pool else {})), data, 11), data


# 0 generated, 1 gather, 2 pattern pass and lists
@pytest.mark.parametrize("spec,routes", [
    ((200, 4, 8, 3), {512: 1, 1024: 1, 2048: 0, 9000: 0}),       # 990 entries in a column, lists of 2000
    ((40, 6, 8), {512: 1, 800: 1, 1024: 0}),                     # lists of 2700
    ((20, 6, 127), {1: 1, 600: 1, 1024: 2, 7000: 2, 8192: 0}),
    ((1, 6, 127), {200: 1, 5000: 2}),                            # little work, many blocks
    ((10, 4, 8), {5000: 1, 20000: 2}),
], ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else "")
def test_interaction_routes(wdf, ctx, spec, routes):
    ens, data = _model(*spec)
    F, most = spec[2], max(routes)
    X = torch.from_numpy(synth.make_matrix(data, most + 9, 4)).cuda()
    bg, gen = (wdf.Background(wdf.Model(ctx, ens, k), X[:, :999].contiguous(), values=wdf.SHAPLEY_IV)
               for k in (wdf.KERNEL_SPECIALISED, wdf.KERNEL_GENERIC))
    assert bg.specialised and not gen.specialised
    assert gen.explain_route(most) == wdf.ROUTE_LISTED
    ref = gen.explain_iv(X)
    for n, route in routes.items():
        assert bg.explain_route(n) == route, n
        assert torch.equal(bg.explain_iv(X[:, 7:7 + n]), ref[:, :, 7:7 + n]), n
    rows = [0, most // 3, most + 8]
    exact = oracle.bg_iv_walk(oracle.Model(ens), np.ascontiguousarray(X[:, rows].cpu().numpy()),
                              np.ascontiguousarray(X[:, :999].cpu().numpy()), threads=8)
    err = np.abs(ref[:, :, rows].cpu().numpy() - exact).max(axis=(0, 1)) / np.abs(exact).max(axis=(0, 1))
    assert err.max() <= 1e-5

"""What a model without generated kernels pays for before its first values: the
load plans its walks and nothing for the LDS, and a summary holds its tables
once."""
import time

import pytest

from paper_2511_09376_amd import synth

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def uneven():
    from paper_2511_09376_amd import wdf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = synth.WORKLOADS["uneven"]
    return wdf, wdf.Context(0), w, w.ensemble()


def test_generic_load_time(uneven):
    """500 uneven trees: 6.6 ms, 2.3 of them layout and coefficient matrices;
    with the search for LDS folds it was 31 ms.  The bound is half of that."""
    wdf, ctx, w, ens = uneven
    best = float("inf")
    for _ in range(6):
        t = time.perf_counter()
        model = wdf.Model(ctx, ens, wdf.KERNEL_GENERIC)
        best = min(best, time.perf_counter() - t)
        model.close()
    print(f"generic load {1e3 * best:.1f} ms", flush=True)
    assert best < 15.5e-3

"""CPU check of the generated explain kernel's stage copies: stage 0 whole, the
others by quarters of the waves, together every 16-byte piece of the explain
tables exactly once, and the loop of the waves without rows the same pieces."""
import re

import numpy as np
import pytest

from paper_2511_09376_amd import synth


@pytest.mark.parametrize("which", ["mid", "uneven"])
def test_stage_copies_cover_the_tables(which):
    from paper_2511_09376_amd import wdf
    w = synth.WORKLOADS[which]
    spec = w.model if which == "mid" else synth.ModelSpec(60, 1, 8, 0.15, 127)
    src = wdf.specialised_source(synth.make_ensemble(spec, w.data, w.seeds()[0]))
    nt = int(re.search(r"#define NT (\d+)", src).group(1))
    tab = int(re.search(r"#define TAB_BYTES (\d+)", src).group(1))
    nq = nt // 4
    copied = np.zeros(tab // 16, np.int32)
    for guard, ofs, c in re.findall(r"(?:if \(threadIdx\.x < (\d+)u\) )?STAGE_PIECE_B\((\d+)u, d_, (\d+)u\)", src):
        a = int(ofs) // 16 + int(c)
        copied[a: a + (int(guard) if guard else nt)] += 1
    quarters = re.findall(r"if \(quarter == (\d)u\) \{ float\* d_ = lds \+ \d+;([^\n]*) \}\n", src)
    assert quarters
    for _, body in quarters:
        for guard, ofs, c in re.findall(r"(?:if \(qthread < (\d+)u\) )?STAGE_QUARTER\((\d+)u, d_, (\d+)u\)", body):
            threads = int(guard) if guard else nq
            assert int(c) % nq == 0 and 0 < threads <= nq
            a = int(ofs) // 16 + int(c)
            assert a + threads <= copied.size
            copied[a: a + threads] += 1
    assert (copied == 1).all()
    # the loop's stages
    at = [int(x) for x in re.search(r"stage_at\[\] = \{([^}]*)\}", src).group(1).split(",")]
    assert at == sorted(at) and at[0] == 0 and 4 * at[-1] == tab and all(x % 4 == 0 for x in at)
    assert {int(o) for o in re.findall(r"STAGE_QUARTER\((\d+)u, d_", src)} == {4 * x for x in at[1:-1]}

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


def _c_int(expr, **names):
    """A C expression of unsigned numbers (and one conditional) from the source."""
    expr = re.sub(r"\b(\d+)u\b", r"\1", expr).replace("/", "//")
    cond = re.fullmatch(r"(.*?) \? (.*?) : (.*)", expr)
    return eval(f"({cond[2]}) if ({cond[1]}) else ({cond[3]})" if cond else expr, {}, names)


@pytest.mark.parametrize("which", ["mid", "uneven60", "uneven500", "wide"])
def test_waves_without_rows_follow_the_others(which):
    """The loop of the waves past the block's rows: the barriers of the other
    waves' code, and of every stage the pieces that their threads copy there.
    The 500 trees pass in more than 256 stages, which are copied at once; so are
    those of 250 features, whose accumulators do not fit the registers."""
    from paper_2511_09376_amd import wdf
    w = synth.WORKLOADS["mid" if which == "mid" else "uneven"]
    spec = w.model if which != "uneven60" else synth.ModelSpec(60, 1, 8, 0.15, 127)
    if which == "wide":
        spec, data = synth.ModelSpec(40, 6, 6, 0.0, 250), synth.DataSpec(250, False, 0.05)
    else:
        data = w.data
    src = wdf.specialised_source(synth.make_ensemble(spec, data, w.seeds()[0]))
    nt = int(re.search(r"#define NT (\d+)", src).group(1))
    at = [int(x) for x in re.search(r"stage_at\[\] = \{([^}]*)\}", src).group(1).split(",")]
    stages = len(at) - 1
    assert (stages > 256) == (which == "uneven500")
    end = src.index("  } else {\n    for (u32 s = 0;")
    rows, idle = src[src.rindex("  if (live) {\n", 0, end):end], src[end:]
    idle = idle[:idle.index("if (live && row < n)")]
    turns = int(re.search(r"for \(u32 s = 0; s < (\d+)u", idle).group(1))
    assert rows.count("__syncthreads();") == turns == stages
    assert f"if (s + 1u >= {stages}u) continue;" in idle
    loop = re.search(r"for \(u32 c = (.*?); c < (\w+); c \+= (\w+)\)\s+if \(c \+ (\S+) < (\w+)\) STAGE_(\w+)\(", idle)
    c1 = re.search(r"const u32 c1 = (.*?);", idle)
    by_quarters = loop[6] == "QUARTER"
    assert by_quarters == (which not in ("uneven500", "wide")) and bool(c1) == by_quarters
    assert loop[2] == loop[5] == ("c1" if by_quarters else "n16")
    assert loop[4] == ("qthread" if by_quarters else "threadIdx.x")
    step = nt if loop[3] == "NT" else int(loop[3].rstrip("u"))
    # what the waves with rows copy: (stage, quarter) -> pieces of the stage
    live = {}
    if by_quarters:
        for q, body in re.findall(r"if \(quarter == (\d)u\) \{ float\* d_ = lds \+ \d+;([^\n]*) \}\n", rows):
            for guard, ofs, c in re.findall(r"(?:if \(qthread < (\d+)u\) )?STAGE_QUARTER\((\d+)u, d_, (\d+)u\)", body):
                s = at.index(int(ofs) // 4)
                live.setdefault((s, int(q)), set()).update(range(int(c), int(c) + (int(guard) if guard else nt // 4)))
    else:
        for guard, ofs, c in re.findall(r"(?:if \(threadIdx\.x < (\d+)u\) )?STAGE_PIECE_B\((\d+)u, d_, (\d+)u\)", rows):
            s = at.index(int(ofs) // 4)
            live.setdefault((s, 0), set()).update(range(int(c), int(c) + (int(guard) if guard else nt)))
    for s in range(1, stages):
        n16 = (at[s + 1] - at[s]) // 4
        seen = set()
        for q in range(4 if by_quarters else 1):
            end = _c_int(c1[1], n16=n16, quarter=q) if c1 else n16
            start = _c_int(loop[1], n16=n16, quarter=q)
            threads = nt // 4 if by_quarters else nt
            mine = {c + t for c in range(start, end, step) for t in range(threads) if c + t < end}
            assert mine == live.get((s, q), set()), (s, q)
            assert not mine & seen
            seen |= mine
        assert seen == set(range(n16)), s

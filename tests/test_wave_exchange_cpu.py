"""Lanes of one wave that pass values through LDS without a workgroup barrier
order their accesses for the compiler too: __builtin_amdgcn_wave_barrier has no
memory effect, so it stands only inside wave_sync (with the fence), and the
kernels that exchange inside a wave call that between the accesses.  Read from
the sources: reordered accesses could only be seen as a race on the GPU."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_13196_amd", "csrc")


def _code(name):
    text = open(os.path.join(CSRC, name)).read()
    return re.sub(r"//[^\n]*|/\*.*?\*/", "", text, flags=re.S)


def _body(code, head):
    """The function whose definition starts with `head`, braces matched."""
    at = code.index("{", code.index(head))
    depth = 0
    for k in range(at, len(code)):
        depth += {"{": 1, "}": -1}.get(code[k], 0)
        if depth == 0:
            return code[at:k + 1]
    raise AssertionError(head)


def _in_order(text, *parts):
    at = 0
    for p in parts:
        m = re.compile(p).search(text, at)
        assert m, (p, text[at:at + 400])
        at = m.end()


def test_wave_barriers_come_with_a_fence():
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".hip", ".h", ".cpp")):
            continue
        code = _code(name)
        if name == "fgl_wave.h":
            _in_order(_body(code, "void wave_sync()"), "__builtin_amdgcn_fence", "__builtin_amdgcn_wave_barrier")
        else:
            assert "wave_barrier" not in code, name


def test_exchanges_inside_a_wave_are_ordered():
    sky, chains = _code("fgl_sky.hip"), _code("fgl_chains.hip")
    # the fills of the regions' runs: read by all lanes, moved on by one, read again
    place = _body(sky, "void k_sky_regions(")
    place = place[place.index("if (tid >= 64) return;"):]
    _in_order(place, r"\bfor\b", r"= [^;=]*s_cnt\[j\]", r"wave_sync\(\)", r"s_cnt\[j\] =", r"wave_sync\(\)",
              r"\bfor\b")
    # the normals of a direction: written in pairs, read in rows, written again
    _in_order(_body(chains, "void new_step("), r"\bu\[2 \* pr\] =", r"wave_sync\(\)", r"\* u\[k\]",
              r"wave_sync\(\)")
    # a channel group's residuals: one lane reads four lanes', then the next pass
    run = _body(chains, "void k_chain_run(")
    _in_order(run, r"s_r\[[^\]]*\] = ", r"wave_sync\(\)", r"acc = fma\(s_r", r"s_part\[f >> 2\] = acc",
              r"wave_sync\(\)")

"""What the wavefronts of the sampler's scan kernel tell each other through LDS: an array with one place per wavefront is
written again only behind a barrier that follows the last read of the others' places (without one, a wavefront that is held up
reads the second value for the first).  A run on the GPU would hardly ever show a missing one, so the source is read."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_02534_amd", "csrc")


def _scan_kernel():
    """The kernel's text without comments and without branches that end in a return."""
    text = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, "sampler.hip")).read())
    start = text.index("void sampler_scan_kernel(")
    body = text[start:text.index("\n}\n", start)]
    return re.sub(r"\n    if \([^\n]*\{\n(?:(?!\n    \}\n)[\s\S])*?        return;\n    \}\n", "\n", body)


def unsafe_writes(body):
    """Names of arrays written at [wave] while other wavefronts may still read what was there."""
    pending, bad = set(), []
    for m in re.finditer(r"(?P<barrier>lds_barrier\(\)|__syncthreads\(\))|L\.(?P<name>\w+)\[(?P<at>\w+)\](?P<set>\s*=(?!=))?", body):
        if m["barrier"]:
            pending.clear()
        elif m["set"] and m["at"] == "wave" and m["name"] in pending:
            bad.append(m["name"])
        elif not m["set"] and m["at"] != "wave":
            pending.add(m["name"])
    return bad


def test_the_check_itself():
    assert unsafe_writes("L.a[wave] = 1; lds_barrier(); m = L.a[w]; L.a[wave] = 2;") == ["a"]
    assert unsafe_writes("L.a[wave] = 1; lds_barrier(); m = L.a[w]; lds_barrier(); L.a[wave] = 2;") == []


def test_no_wavefront_overwrites_what_others_may_still_read():
    body = _scan_kernel()
    assert "if (greedy)" not in body and "L.red_f[wave]" in body and "L.mass[wave]" in body
    assert unsafe_writes(body) == []

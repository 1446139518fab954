"""Kernels that latch an error go by the status word as a workgroup, not wave by wave.

A launch that latches errors changes the status word while its own workgroups
still start.  Where the waves of a workgroup share LDS, one of them may then not
leave on that word while another goes on: the other one would read LDS that was
never written, cell lists and counts among it.  Read from the sources: which
kernels can latch and have barriers (through any function that they call)."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2208_07412_amd", "csrc")
# barriers that no workgroup of the kernel comes to before its waves part
ALONE = {"k_sample_index": "block_index without LDS: the waves share nothing"}


def close(s, i, pair):
    """The index past the bracket that closes the one at s[i]."""
    depth = 0
    while True:
        depth += {pair[0]: 1, pair[1]: -1}.get(s[i], 0)
        i += 1
        if not depth:
            return i


def functions():
    """name -> (head, body, is a kernel) of every function in the sources."""
    out = {}
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hpp"))):
        s = re.sub(r"//[^\n]*|/\*.*?\*/", "", open(path).read(), flags=re.S)
        for m in re.finditer(r"__(global|device)__", s):
            i = m.end()
            while True:  # to the bracket of the parameters, past those of attributes
                o = re.compile(r"(\w*)\s*\(|;").search(s, i)
                if o.group() == ";" or not o.group(1).startswith("__"):
                    break
                i = close(s, o.end() - 1, "()")
            if o.group() == ";":
                continue
            p = close(s, o.end() - 1, "()")
            b = re.compile(r"\s*(const)?\s*\{").match(s, p)
            if b:
                out[o.group(1)] = (s[m.end():o.start()], s[b.end():close(s, b.end() - 1, "{}")],
                                   m.group(1) == "global")
    return out


FN = functions()


def reached(name, seen=None):
    seen = {name} if seen is None else seen
    for w in set(re.findall(r"\b(\w+)\b", FN[name][1])):
        if w in FN and w not in seen:
            seen.add(w)
            reached(w, seen)
    return seen


def test_waves_leave_together():
    shared = []
    for name, (head, _, kernel) in FN.items():
        threads = re.search(r"__launch_bounds__\(([^,)]+(\* NW)?)", head)
        if not kernel or (threads and threads.group(1).strip() == "64"):
            continue  # one wave
        fns = reached(name)
        body = "".join(FN[f][1] for f in fns if f not in ("failed_wg",))
        if "latch" in fns and "__syncthreads" in body:
            shared.append(name)
    # the kernels that the rule is about are found
    assert {"k_cluster_peaks_mw", "k_cm_track_bits", "k_cm_dec_tracks", "k_hit_grid",
            "k_zs_decode"} <= set(shared), shared
    wrong = [n for n in shared if n not in ALONE and
             (re.search(r"\bfailed\(", FN[n][1]) or "failed_wg(" not in FN[n][1])]
    assert not wrong, wrong

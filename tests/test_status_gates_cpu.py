"""Gates of the check kernels, read from the sources.

A kernel that returns early when an input check has failed, raises such bits
itself and has workgroup barriers must not gate on the bits it raises: its
other workgroups set them while it runs, and a workgroup of which only some
waves see the bit would go on with shared memory that was never filled.
(A launch of a single workgroup raises its bits after its waves have read the
word.)
"""

import glob
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2010_14058_amd", "csrc")


def _sources():
    return {os.path.basename(p): open(p).read() for p in sorted(glob.glob(CSRC + "/*.h*"))}


def _input_bits(src):
    bits = {m[1]: m[2] for m in re.finditer(r"(ST_\w+) = 1u << (\d+)", src)}
    expr = re.search(r"ST_INPUT\s*=\s*([^;]*);", src)[1]
    return bits, set(re.findall(r"ST_\w+", expr))


def _kernels(sources):
    for name, src in sources.items():
        src = re.sub(r"//[^\n]*", "", src)
        for part in re.split(r"(?=__global__)", src)[1:]:
            body = part[:part.find("\n}\n")]
            k = re.search(r"\b(k_\w+)\s*\(", body)
            if k:
                yield name, k[1], body, src


def _gate_ignores(body, all_input):
    """Input bits the kernel's early return does not look at (None: no gate)."""
    m = re.search(r"failed_before\([^,]+,\s*([^;]*?)\)\)\s*return", body)
    if m:
        expr = m[1]
        if "~" in expr:
            keep = set(re.findall(r"ST_\w+", expr.split("~", 1)[1]))
            return all_input - keep
        return set(re.findall(r"ST_\w+", expr))
    if "input_failed(" in body or re.search(r"load_agent\(status\)[^;]*return", body):
        return set()
    return None


def test_kernels_with_barriers_do_not_gate_on_their_own_bits():
    sources = _sources()
    _, all_input = _input_bits(sources["tg_internal.hpp"])
    seen = []
    for name, kernel, body, src in _kernels(sources):
        if not ("__syncthreads" in body or "slot_tile(" in body):
            continue
        raised = {b for b in re.findall(r"\bST_\w+", re.sub(r"failed_before\([^;]*;", "", body))
                  if b in all_input}
        ignores = _gate_ignores(body, all_input)
        if not raised or ignores is None:
            continue
        if re.search(kernel + r"<<<1,", src):
            continue
        seen.append(kernel)
        assert raised <= ignores, f"{name}: {kernel} gates on {sorted(raised - ignores)}"
    assert {"k_check_slots", "k_slot_keys", "k_dir_slots", "k_small_check"} <= set(seen)


@pytest.mark.parametrize("name,func", [("tg_api.hip", "status_from_bits"),
                                       ("tg_kernels.hip", "k_status_code")])
def test_every_input_bit_has_a_status(name, func):
    sources = _sources()
    _, all_input = _input_bits(sources["tg_internal.hpp"])
    src = sources[name]
    body = src[src.index(func + "("):]
    body = body[:body.index("\n}\n")]
    assert all_input <= set(re.findall(r"\bST_\w+", body))

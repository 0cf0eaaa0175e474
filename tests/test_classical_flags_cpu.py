"""The classical iteration's kernels leave early when a flag in device memory says that both systems
have converged, ahead of workgroup barriers: all waves of a workgroup have to read the same value, so
no kernel of several workgroups may write a flag that it leaves by. Read from the source: the flags
that each kernel tests before a return, against the members that it, or a function it calls, writes."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2601_10057_amd", "csrc")
ONE_WORKGROUP = {"k_cl_last"}      # launched with one workgroup, its flag written behind a barrier


def functions():
    """{name: body} of the functions and kernels of the file."""
    src = open(os.path.join(CSRC, "classical_kernels.hpp")).read()
    src = re.sub(r"//[^\n]*", "", src)
    src = re.sub(r"__launch_bounds__\([^()]*(?:\([^()]*\))?[^()]*\)", "", src)
    out = {}
    for m in re.finditer(r"(\w+)\s*\(([^;{}]*)\)\s*\{", src):
        head = src[:m.start()].rsplit(";", 1)[-1].rsplit("}", 1)[-1]
        if "__global__" not in head and "__device__" not in head:
            continue
        depth, end = 1, m.end()
        while depth:
            depth += {"{": 1, "}": -1}.get(src[end], 0)
            end += 1
        out[m.group(1)] = src[m.end():end]
    return out


def written(name, fns):
    body = fns[name]
    w = set(re.findall(r"sc->(\w+)(?:\[[^=;]*\])?\s*(?:[+\-*/|&]?=)(?!=)", body))
    for other in fns:
        if other != name and re.search(r"\b%s\b\s*(?:<[^;()]*>)?\(" % other, body):
            w |= written(other, fns)
    return w


def left_by(body):
    """Members read by the conditions of returns, directly or through a local constant."""
    local = dict(re.findall(r"const int (\w+) = sc->(\w+);", body))
    out = set()
    for cond in re.findall(r"if \(([^;{}]*)\) return;", body):
        out |= set(re.findall(r"sc->(\w+)", cond))
        out |= {local[v] for v in re.findall(r"\b\w+\b", cond) if v in local}
    return out


def test_no_kernel_writes_a_flag_that_it_leaves_by():
    fns = functions()
    kernels = {n for n in fns if n.startswith("k_cl_")}
    assert {"k_cl_matvec", "k_cl_update_rows", "k_cl_inv_rows", "k_cl_last"} <= kernels
    leaving = {n: left_by(fns[n]) for n in kernels}
    assert leaving["k_cl_matvec"] and leaving["k_cl_update_rows"] and leaving["k_cl_inv_rows"]
    for n in kernels - ONE_WORKGROUP:
        both = leaving[n] & written(n, fns)
        assert not both, (n, both)
    # and the test of convergence is made in the kernel that the others follow
    assert "done_all" in written("k_cl_inv_rows", fns)

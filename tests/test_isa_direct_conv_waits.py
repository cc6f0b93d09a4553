"""Waits of the direct convolution's staged patches, and of every barrier behind an access to LDS, read off the compiler's assembly (no GPU).

The patch kernel waits for counts of loads: for the patch with the weights' loads behind it in flight, for a step's weights with those of
the steps after it in flight, for a step's pixels with those of the next step in flight.  That holds only while the compiler leaves the
loads in the order of the source, and it gains something only while it adds no full wait of its own.  A barrier stands for "everybody has
read this buffer" only where the reads before it have returned."""
import re

import pytest

import paper_2007_12216_amd as rn
from test_isa_wait_states import functions


def in_flight_at_barriers(code, labels):
    """[(access to LDS, barrier's index)]: accesses that may be in flight when a wave meets a barrier."""
    found = []
    for at, (op, _, _, text) in enumerate(code):
        if not op.startswith("ds_"):
            continue
        paths, seen = [(at + 1, 0)], {}                   # accesses after this one: they return in order
        while paths:
            i, later = paths.pop()
            if i >= len(code) or seen.get(i, 1 << 30) <= later:
                continue
            seen[i] = later
            op2, operands, _, text2 = code[i]
            wait = re.search(r"lgkmcnt\((\d+)\)", text2) if op2 == "s_waitcnt" else None
            if op2 == "s_endpgm" or (wait and int(wait.group(1)) <= later):
                continue
            if op2 == "s_barrier":
                found.append((text, i))
                continue
            if op2 == "s_branch" or op2.startswith("s_cbranch"):
                paths.append((labels[operands[0]], later))
            if op2 != "s_branch":
                paths.append((i + 1, later + op2.startswith("ds_")))
    return found


def test_the_walk_sees_a_barrier_that_does_not_wait(tmp_path):
    # the read at the loop's end is in flight where the loop begins again
    text = "_Zplanted:\n\tds_write_b32 v0, v1\n\ts_waitcnt lgkmcnt(0)\n.L1:\n\t%s\n\ts_barrier\n\tds_read_b128 v[0:3], v8\n\ts_cbranch_scc1 .L1\n\ts_endpgm\n"
    for wait, bad in (("s_nop 0", 1), ("s_waitcnt vmcnt(0)", 1), ("s_waitcnt lgkmcnt(1)", 1), ("s_waitcnt vmcnt(3) lgkmcnt(0)", 0)):
        path = tmp_path / "planted.s"
        path.write_text(text % wait)
        (code, labels), = functions(path).values()
        assert len(in_flight_at_barriers(code, labels)) == bad


def test_every_access_to_lds_is_done_before_a_barrier(assembly):
    found = {name: v for name, (code, labels) in assembly.items() for v in [in_flight_at_barriers(code, labels)] if v}
    assert not found, "\n".join(f"{name}: {v[0]} ({len(v)} in all)" for name, v in found.items())


def count(text, counter):
    found = re.search(counter + r"\((\d+)\)", text)
    return int(found.group(1)) if found else 1 << 30


@pytest.mark.parametrize("variant", [v for v in rn.rnswino_direct_variants() if v.startswith("k_direct_conv_patch")])
def test_the_patch_kernel_counts_the_loads_it_means(assembly, variant):
    numbers = re.findall(r"\d+", variant.partition("<")[2])
    _, _, RM, NT, D = map(int, numbers)
    name, = [n for n in assembly if "k_direct_conv_patchI" + "".join(f"Li{n}E" for n in numbers) in n]
    code = [(op, text) for op, _, _, text in assembly[name][0]]
    ops = [op for op, _ in code]

    def weights(lo, hi):
        return ops[lo:hi].count("global_load_dwordx4")

    # before the first barrier: the patch, all D sets of weights in the order of the steps, the wait that leaves these in flight
    barrier = ops.index("s_barrier")
    patch = max(i for i in range(barrier) if ops[i] == "global_load_lds_dwordx4")
    wait = max(i for i in range(barrier) if ops[i] == "s_waitcnt" and "vmcnt" in code[i][1])
    assert count(code[wait][1], "vmcnt") == RM * D == weights(patch, wait) == weights(0, wait) and weights(wait, barrier) == 0
    # the D steps of the loop: next pixels read; no wait for these, nor for the weights of later steps; RM loads of weights, in front of
    # whatever the next step waits for at a new channel block
    at = ops.index("ds_read_b128")
    for d in range(D):
        product = next(i for i in range(at, len(ops)) if ops[i].startswith("v_mfma"))
        read = max(i for i in range(product) if ops[i] == "ds_read_b128")
        following = next(i for i in range(product, len(ops)) if ops[i] == "ds_read_b128")
        last = max(i for i in range(following) if ops[i] == "global_load_dwordx4")
        assert weights(read, following) == RM and not any(op.startswith("v_mfma") for op in ops[last:following])
        for i in range(read, last):
            if ops[i] == "s_waitcnt":
                assert count(code[i][1], "lgkmcnt") >= NT and count(code[i][1], "vmcnt") >= RM * (D - 1), (d, code[i][1])
        boundary = range(at, min(j for j in range(at, product) if ops[j] == "s_barrier"))
        assert [count(code[i][1], "vmcnt") for i in boundary if ops[i] == "s_waitcnt" and "vmcnt" in code[i][1]] == [3 * RM], d
        at = last


def test_a_single_tap_never_takes_a_patch():
    for N, C, K, hw in ((1, 64, 16, 7), (1, 640, 64, 14), (8, 256, 256, 28), (8, 64, 1024, 56), (8, 2048, 512, 7)):
        assert rn.rnswino_direct_describe(N, C, K, hw, hw, 1, 0)["kernel"].startswith("k_direct_conv<")

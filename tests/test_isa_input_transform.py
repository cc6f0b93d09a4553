"""What the one-tile input transform fetches, read off the compiler's assembly (no GPU): its arguments all at entry.  An argument fetched
after the gather's loads stands between them and the first table load, a wait of about 500 cycles in the first kernel of a layer."""
import re

import pytest

import paper_2007_12216_amd as rn


@pytest.mark.parametrize("variant", [v for v in rn.rnswino_kernel_variants() if v.startswith("k1_input_transform<") and not v.endswith("true>")])
def test_no_argument_is_fetched_between_the_gather_and_the_table(assembly, variant):
    KS1, wide, _ = variant.partition("<")[2].rstrip(">").split(", ")
    name, = [n for n in assembly if f"k1_input_transformILi{KS1}ELb{int(wide == 'true')}ELb0EEE" in n]
    ops = [op for op, _, _, _ in assembly[name][0]]
    gather = ops.index("global_load_dwordx4")
    stored = next(i for i in range(gather, len(ops)) if ops[i].startswith("ds_write"))
    loads = [i for i in range(gather, stored) if ops[i] == "global_load_dwordx4"]
    assert len(loads) > int(KS1)                            # the table's first fragments are requested here too
    assert not any(op.startswith("s_load") for op in ops[gather:loads[-1]])


def test_the_layer_kernels_take_few_arguments(assembly_file):
    """A launch of up to 112 bytes of arguments takes the host three quarters of the time of one of 120 and more."""
    text = open(assembly_file).read()
    sizes = {name: int(size) for size, name in re.findall(r"\.kernarg_segment_size:\s+(\d+)(?:(?!\.kernarg_segment_size).)*?\.name:\s+(_Z\w+)", text, re.S)}
    layer = {n: s for n, s in sizes.items() if any(k in n for k in ("k1_input", "k2_residue", "k12_transform", "k3_inverse"))}
    assert len(layer) == len(rn.rnswino_kernel_variants()) and max(layer.values()) <= 112, layer

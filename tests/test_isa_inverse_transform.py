"""Registers of the inverse transform over 16-bit moduli, read off the compiler's metadata (no GPU): its loads, products and binary64
arithmetic follow each other, so that a wave per SIMD less takes up to twice as long.  And of the one over 8-bit moduli, read off the assembly, that
the divisions of a lane's position are done while its loads are in flight, where these are few."""
import pytest

import paper_2007_12216_amd as rn

REGISTERS = 512                     # of a SIMD, for all its waves
WAVES = {1: (8, 8, 6, 5), 2: (6, 4, 3, 2), 3: (4, 3, 4, 3), 4: (3, 2, 2, 2), 5: (3, 3, 2, 2), 6: (2, 2, 2, 1), 7: (2, 2, 2, 1), 8: (2, 2, 1, 1)}


@pytest.mark.parametrize("moduli,steps", [(n, s) for n in WAVES for s in (1, 2, 3, 4)])
def test_waves_per_simd(vector_registers, moduli, steps):
    count, = [v for k, v in vector_registers.items() if f"14k3_inverse_crtILi{moduli}ELi{steps}ELb1E" in k]
    assert REGISTERS // (-(-count // 8) * 8) >= WAVES[moduli][steps - 1], count


@pytest.mark.parametrize("variant", [v for v in rn.rnswino_kernel_variants() if v.startswith("k3_inverse_crt<") and v.split(", ")[2] == "false" and
                                     int(v[15]) * int(v[18]) <= 8])
def test_the_position_is_known_before_the_barrier(assembly, variant):
    moduli, steps, _, fast = variant.partition("<")[2].rstrip(">").split(", ")
    name, = [n for n in assembly if f"14k3_inverse_crtILi{moduli}ELi{steps}ELb0ELb{int(fast == 'true')}E" in n]
    ops = [op for op, _, _, _ in assembly[name][0]]
    divisions = [i for i, op in enumerate(ops) if op == "v_mul_hi_u32"]
    first, barrier = ops.index("global_load_dword"), ops.index("s_barrier")
    assert len(divisions) >= 3 and all(i < barrier for i in divisions) and sum(i > first for i in divisions) >= 2

"""Registers of the inverse transform over 16-bit moduli, read off the compiler's metadata (no GPU): its loads, products and binary64
arithmetic follow each other, so that a wave per SIMD less takes up to twice as long."""
import pytest

REGISTERS = 512                     # of a SIMD, for all its waves
WAVES = {1: (8, 8, 6, 5), 2: (6, 4, 3, 2), 3: (4, 3, 4, 3), 4: (3, 2, 2, 2), 5: (3, 3, 2, 2), 6: (2, 3, 2, 1), 7: (2, 2, 2, 1), 8: (2, 2, 1, 1)}


@pytest.mark.parametrize("moduli,steps", [(n, s) for n in WAVES for s in (1, 2, 3, 4)])
def test_waves_per_simd(vector_registers, moduli, steps):
    count, = [v for k, v in vector_registers.items() if f"14k3_inverse_crtILi{moduli}ELi{steps}ELb1E" in k]
    assert REGISTERS // (-(-count // 8) * 8) >= WAVES[moduli][steps - 1], count

"""Host-side checks of the kernel selection (no GPU): the layers of tests/variant_cases.py reach every instantiation the
library can launch, the conversion out of the RNS takes the expected form at the edges the GPU parity cases sit on, and no
admissible moduli set is left without an instantiation."""
import itertools

import pytest

import paper_2007_12216_amd as rn
import variant_cases as vc

HOST = rn.FLAG_HOST_ONLY
UNCHECKED = rn.FLAG_ALLOW_UNCHECKED_RANGE


def test_the_variant_cases_reach_every_instantiation():
    kept = vc.select_cases()
    reached = {k for _, kernels, _ in kept for k in kernels}
    every = {k for k in rn.rnswino_kernel_variants() if not k.startswith("k12_transform_gemm")}      # (that one: test_gpu_transform_gemm.py)
    assert len(every) > 100
    assert every - reached == set(), sorted(every - reached)
    assert reached - every == set()
    assert {c for _, _, c in kept} == {"unreduced-binary32", "unreduced-binary64", "reduced-binary32", "reduced-binary64",
                                       "reduced-binary64-mul32"}
    # the streaming inverse transform in all its output modes, with each conversion it can take
    stream = {(c, case[10]) for case, kernels, c in kept if kernels[2].startswith("k3_inverse_crt_stream")}
    assert stream >= {(c, mode) for c in ("unreduced-binary32", "unreduced-binary64", "reduced-binary32") for mode in (0, 1, 2)}
    # and the whole list stays affordable for the CPU oracle: direct-convolution operations of all cases together
    gop = sum(2.0 * c[0] * c[1] * c[2] * c[3] * c[4] * c[5] ** 2 for c, _, _ in kept) / 1e9
    assert gop < 600.0


def test_the_direct_convolution_cases_reach_every_instantiation():
    from test_gpu_direct import CASES
    reached = {}
    for case in CASES:
        reached.setdefault(rn.rnswino_direct_describe(*case)["kernel"], []).append(case)
    assert sorted(reached) == sorted(rn.rnswino_direct_variants())
    # staged patches of 256 pixels, also with the last row block shifted back (its rows are then stored by two blocks)
    for kernel, rm in (("k_direct_conv_patch<1, 4, 2, 4, 4>", 2), ("k_direct_conv_patch<1, 4, 4, 4, 4>", 4)):
        assert any(-(-case[2] // 16) % rm for case in reached[kernel])
        assert {case[1] > 64 for case in reached[kernel]} == {True, False}       # one channel block, and the two buffers
    for bad, code in (((1, 4, 4, 2, 2, 5, 0), -1), ((1, 1 << 20, 4, 8, 8, 3, 1), -2), ((1, 4, 4, 8, 8, 17, 8), -2)):
        with pytest.raises(rn.RnsWinoError) as e:
            rn.rnswino_direct_describe(*bad)
        assert e.value.code == code


def test_the_filter_transform_cases_fill_the_fragments_of_every_instantiation():
    """k0_filter_transform<width, PP>: a filter takes PP = 1, 2 or 4 of a fragment's four slices, the fragment 4 / PP channels."""
    from test_gpu_filter_transform import CASES
    reached = set()
    for C, K, r, m, moduli, T in CASES:
        pieces = (r * r + 15) // 16
        if C >= 64:
            reached.add((moduli[0] > 255, 4 if pieces > 2 else pieces))
    assert reached == {(wide, pp) for wide in (False, True) for pp in (1, 2, 4)}


@pytest.mark.parametrize("case,patches", [
    ((1, 2048, 512, 7, 7, 1, 0), False), ((8, 64, 64, 56, 56, 1, 0), False),                  # a single tap
    ((8, 3, 512, 112, 112, 3, 1), False), ((8, 128, 256, 112, 112, 3, 1), False),             # few steps, many blocks
    ((8, 64, 256, 56, 56, 3, 1), True), ((8, 129, 256, 112, 112, 3, 1), True), ((8, 64, 64, 224, 224, 3, 1), True),
    ((8, 64, 256, 28, 28, 2, 1), False), ((8, 64, 1024, 28, 28, 2, 1), False),                # 2 x 2 filters
    ((8, 64, 64, 28, 28, 2, 1), True), ((8, 64, 1024, 56, 56, 2, 1), True), ((8, 256, 1024, 28, 28, 2, 1), True),
    ((8, 256, 256, 56, 56, 3, 1), True), ((1, 3, 8, 7, 7, 3, 1), True)])
def test_the_direct_convolution_stages_patches_only_where_they_are_used_often_enough(case, patches):
    """Both sides of each line, measured (times beside choose_direct); with patches the 1 x 1 layers took up to 1.5 times as long."""
    assert rn.rnswino_direct_describe(*case)["kernel"].startswith("k_direct_conv_patch") == patches


@pytest.mark.parametrize("n,N,C,hw,r,m,sixteen", [
    (4, 12, 128, 14, 5, 4, True), (2, 4, 128, 35, 3, 4, False), (1, 4, 128, 56, 3, 4, True),            # t <= 8
    (4, 4, 128, 112, 3, 8, True), (1, 8, 64, 112, 3, 8, True), (4, 8, 64, 224, 3, 8, True),             # t = 9, 10: 384 blocks
    (4, 6, 256, 56, 3, 8, False), (4, 6, 128, 56, 3, 8, False), (1, 7, 256, 56, 3, 8, False),
    (4, 1, 128, 112, 3, 8, True), (3, 1, 128, 112, 3, 8, False), (4, 8, 64, 56, 3, 8, True),            # few blocks of one tile
    (3, 24, 256, 28, 3, 8, True), (2, 21, 256, 35, 3, 8, False), (4, 32, 512, 28, 3, 8, True),          # planes below 49 tiles
    (4, 320, 128, 8, 3, 8, False), (3, 1600, 128, 8, 3, 8, False), (4, 1100, 256, 8, 3, 8, True),       # planes of one tile
    (8, 12, 64, 14, 5, 4, False), (8, 24, 64, 14, 5, 4, True),                                          # many moduli, 48 and 96 blocks
    (4, 1, 256, 56, 3, 8, False), (1, 1, 16, 16, 3, 8, False)])
def test_the_input_transform_takes_16_tiles_at_a_time_only_where_that_is_faster(n, N, C, hw, r, m, sixteen):
    """Both sides of each line, measured (times beside the rule); on the layers of one tile per plane 16 tiles took up to 1.3 times as long."""
    plan = rn.rnswino_plan(N, C, 64, hw, hw, r, m, r // 2, (251, 241, 239, 233, 229, 227, 223, 211)[:n], flags=HOST | UNCHECKED)
    assert rn.rnswino_plan_describe(plan)["kernels"][0].startswith("k1_input_transform_tiles") == sixteen


@pytest.mark.parametrize("N,C,K,hw,r,m,moduli,grid", [
    (1, 128, 128, 28, 5, 12, (251, 241, 239, 233), "grid=24x4x2"), (1, 512, 512, 28, 3, 14, (65521, 65519), "grid=32x2x2"),
    (1, 20, 3, 20, 3, 10, (251, 241, 239), "grid=8x3x2"), (1, 20, 3, 18, 3, 9, (251, 241, 239), "grid=8x3"),               # 9 column blocks, 8
    (2, 128, 3, 56, 3, 14, (65521, 65519), "grid=64x2x2"), (2, 192, 3, 56, 3, 14, (65521, 65519), "grid=96x2"),            # 128 blocks, 192
    (1, 128, 3, 28, 5, 12, (251,), "grid=24x1"), (8, 512, 3, 224, 3, 14, (251, 241), "grid=16384x1")])                     # all residues in a block
def test_the_report_tells_which_input_transforms_share_column_blocks(N, C, K, hw, r, m, moduli, grid):
    plan = rn.rnswino_plan(N, C, K, hw, hw, r, m, r // 2, moduli, flags=HOST | UNCHECKED)
    assert rn.rnswino_plan_describe(plan)["grids"][0] == grid


def _conversion(C, moduli, r=3, m=8, flags=HOST, K=16, hw=16):
    plan = rn.rnswino_plan(1, C, K, hw, hw, r, m, r // 2, moduli, flags=flags)
    return rn.rnswino_plan_describe(plan)["conversion"]


def test_conversion_form_at_the_edges_the_gpu_cases_sit_on():
    """Which form of the conversion out of the RNS (section 3) a layer takes is decided on the host from its worst case
    2^14 r^2 C against the product of the moduli; the GPU parity cases at the edge of the dynamic range rely on these."""
    three, four = (251, 241, 239), (251, 241, 239, 233)
    assert _conversion(16, three) == "unreduced-binary32"
    assert _conversion(42, three) == "unreduced-binary32"       # largest C with room for the binary32 error bound
    assert _conversion(43, three) == "unreduced-binary64"
    assert _conversion(49, three) == "unreduced-binary64"       # the edge of the range of three moduli
    assert _conversion(50, three, flags=HOST | UNCHECKED) == "unreduced-binary64"
    assert _conversion(256, four) == "unreduced-binary32"       # the VGG16-style layer
    assert _conversion(11422, four) == "unreduced-binary64"     # the edge of the range of four moduli
    assert _conversion(512, three, flags=HOST | UNCHECKED) == "unreduced-binary64"     # the paper's setting, range trusted
    # four moduli near 253: two quotients are closer than the binary64 sum of unreduced accumulators resolves
    assert _conversion(9800, (253, 251, 247, 241), flags=HOST | UNCHECKED) == "reduced-binary32"      # |y| <= 0.45 P
    assert _conversion(11600, (253, 251, 247, 241), flags=HOST | UNCHECKED) == "reduced-binary64"
    assert _conversion(64, (253, 251, 247, 241)) == "unreduced-binary32"
    # five and more moduli: a partial product P/p_i no longer fits 24 bits
    assert _conversion(64, (251, 241, 239, 233, 229)) == "reduced-binary64-mul32"
    # 16-bit moduli always reduce (their accumulators are three byte-plane sums)
    assert _conversion(512, (65521, 65519), m=14) == "reduced-binary32"
    assert _conversion(14000, (65521, 65519), m=14) == "reduced-binary64"
    assert _conversion(16, (65521, 65519, 65497), m=14) == "reduced-binary64-mul32"


def test_workload_kernels():
    """The instantiations the five benchmark workloads launch (the names a kernel trace of bench.py shows)."""
    import synth_inputs as si
    want = {1: ("k1_input_transform<2, false, false>", "k2_residue_gemm<1, 1, 2, false>", "k3_inverse_crt<3, 2, false, true>"),
            2: ("k1_input_transform<2, false, false>", "k2_residue_gemm_lds<4, 1, 2, 4, 4>", "k3_inverse_crt<4, 2, false, true>"),
            3: ("k1_input_transform<4, false, false>", "k2_residue_gemm<2, 1, 2, false>", "k3_inverse_crt<4, 4, false, true>"),
            4: ("k1_input_transform<4, true, false>", "k2_residue_gemm<4, 1, 2, true>", "k3_inverse_crt<2, 4, true, false>")}
    for idx, kernels in want.items():
        c = si.layer_config(idx)
        plan = rn.rnswino_plan(c["N"], c["C"], c["K"], c["H"], c["W"], c["r"], c["m"], c["pad"], c["moduli"], flags=HOST)
        assert tuple(rn.rnswino_plan_describe(plan)["kernels"]) == kernels, idx


@pytest.mark.parametrize("t", [13, 14, 15, 16])
def test_every_admissible_set_of_four_moduli_has_an_instantiation(t):
    """With 13 and more interpolation points the reduced conversion has no instantiation for exactly four 8-bit moduli
    (no admissible set's product is large enough to need it): every such set must still give a plan, whatever the
    channel count."""
    r, m = 3, t - 2
    ok = [p for p in range(129, 254, 2) if rn_accepts(p, r, m)]
    top = sorted(ok)[-7:]
    tried = 0
    for moduli in itertools.combinations(top, 4):
        try:
            plan = rn.rnswino_plan(1, 12000, 8, m, m, r, m, 1, moduli, flags=HOST | UNCHECKED)
        except rn.RnsWinoError as e:
            assert e.code == -3, (moduli, e.code)       # not pairwise coprime: refused for that reason only
            continue
        assert rn.rnswino_plan_describe(plan)["conversion"].startswith("unreduced")
        tried += 1
    assert tried >= 10


def rn_accepts(p, r, m):
    try:
        rn.rnswino_plan(1, 1, 1, m, m, r, m, 1, (p,), flags=HOST | UNCHECKED)
    except rn.RnsWinoError:
        return False
    return True


def test_16_bit_moduli_refuse_contractions_of_1024_steps():
    """Three unreduced 32-bit byte-plane sums: the middle one gains up to 2^21 per 64-channel step."""
    def code(C):
        try:
            rn.rnswino_plan(1, C, 4, 4, 4, 1, 4, 0, (65521, 65519), flags=HOST | UNCHECKED)
        except rn.RnsWinoError as e:
            return e.code
        return 0
    assert code(65472) == 0 and code(65473) == -2
    assert code(131071) == -2


def test_measurement_flag_selects_the_64_by_16_gemm_blocks():
    plain = rn.rnswino_plan(8, 64, 64, 56, 56, 3, 8, 1, (251, 241, 239, 233), flags=HOST)
    forced = rn.rnswino_plan(8, 64, 64, 56, 56, 3, 8, 1, (251, 241, 239, 233), flags=HOST | rn.FLAG_GEMM_BLOCK_64X16)
    assert rn.rnswino_plan_describe(plan=plain)["kernels"][1] == "k2_residue_gemm<1, 4, 2, false>"
    assert rn.rnswino_plan_describe(plan=forced)["kernels"][1] == "k2_residue_gemm_lds<4, 1, 1, 1, 4>"
    wide = rn.rnswino_plan(1, 64, 64, 28, 28, 3, 14, 1, (65521, 65519), flags=HOST | rn.FLAG_GEMM_BLOCK_64X16)
    assert rn.rnswino_plan_describe(plan=wide)["kernels"][1].startswith("k2_residue_gemm<")      # 8-bit moduli only

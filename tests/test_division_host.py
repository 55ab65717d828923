"""Which division of the work the shapes of the GPU tests take, by the host rules of the library (no GPU needed): a test that is
meant for a kernel's own loop must not be served by a key split, and the other way round, whatever becomes of the rules."""
import ctypes
import os
import shutil
import subprocess

import pytest

import test_tiles_gpu
from paper_2407_08608_amd import binding

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    lib = str(tmp_path_factory.mktemp("division") / "query.so")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "division", "query.cpp"), "-o", lib],
                   check=True, stderr=subprocess.DEVNULL)
    lib, ci, cl = ctypes.CDLL(lib), ctypes.c_int, ctypes.c_long
    lib.key_split.argtypes = [ci, cl, ci, ci, ci]
    lib.backward_form.argtypes, lib.backward_form.restype = [cl, cl, ci, ci, ci], ctypes.c_char_p
    lib.backward_own_row_sums.argtypes = [cl, cl, ci, ci]
    return lib


@pytest.fixture(scope="module")
def key_split(rules):
    return lambda fp8, heads, N, d, causal: bool(rules.key_split(int(fp8), heads, N, d, int(causal)))


@pytest.fixture(scope="module")
def backward_form(rules):
    return lambda heads, kv_heads, N, d, causal: rules.backward_form(heads, kv_heads, N, d, int(causal)).decode()


@pytest.fixture(scope="module")
def own_row_sums(rules):
    return lambda heads, kv_heads, N, d: bool(rules.backward_own_row_sums(heads, kv_heads, N, d))


def _parameters(test, *names):
    """The cases of a parametrised test, as tuples of the named parameters (of one decorator)."""
    for mark in test.pytestmark:
        if mark.name == "parametrize":
            have = mark.args[0].split(",")
            if set(names) <= set(have):
                return [tuple(c[have.index(n)] for n in names) for c in mark.args[1]]
    raise AssertionError(names)


def test_main_loops_are_the_kernels_they_are_meant_for(key_split):
    for fp8, d, causal, N, H, kernel in test_tiles_gpu.MAIN_LOOPS:
        assert not key_split(fp8, H, N, d, causal), (fp8, d, causal, N, H)
        name = binding.fa_fwd_kernel_name(binding.FA_FP8_E4M3 if fp8 else binding.FA_BF16, N, d, causal)
        assert name.startswith(kernel), (fp8, d, causal, N, name)


def test_tests_of_whole_tiles_make_no_key_split(key_split):
    for fp8, d, causal, N, B, H, H_kv in test_tiles_gpu.SHARED_HEADS:
        assert not key_split(fp8, B * H, N, d, causal), (fp8, d, causal, N, B, H)
    for d, N, H in _parameters(test_tiles_gpu.test_forward_shared_tiles, "d", "N", "H"):
        assert not key_split(False, H, N, d, False) and not key_split(False, H, N, d, True), (d, N, H)
    for d, causal, N, H in _parameters(test_tiles_gpu.test_forward_tiles_of_a_head_on_one_xcd, "d", "causal", "N", "H"):
        assert not key_split(False, H, N, d, causal), (d, causal, N, H)


def test_rows_without_an_output_are_tested_in_both_divisions(key_split):
    for dtype, d, N, H in test_tiles_gpu._FORMS_FWD:
        if dtype != "f32":
            assert {key_split(dtype == "fp8", H, N, d, c) for c in (False, True)} == {H == 2}, (dtype, d, N, H)


def test_tests_of_key_splits_make_them(key_split):
    # all but the few shapes whose tiles are too few (FP8 d = 128) or too many (d = 256 without a mask)
    for fp8, test in ((False, test_tiles_gpu.test_forward_with_the_keys_split_over_the_waves),
                      (True, test_tiles_gpu.test_fp8_forward_with_the_keys_split_over_the_waves)):
        for H, N in _parameters(test, "H", "N"):
            split = [(d, c) for d in (64, 128, 256) for c in (False, True) if key_split(fp8, H, N, d, c)]
            assert {(64, False), (64, True)} <= set(split) and len(split) >= 4, (fp8, H, N, split)
    for d, causal, N, heads in _parameters(test_tiles_gpu.test_forward_key_splits_of_four_and_eight_waves, "d", "causal", "N", "heads"):
        assert all(key_split(False, H, N, d, causal) for H in heads), (d, causal, N, heads)


def test_tests_of_the_key_split_rule_lie_on_both_sides_of_it(key_split):
    for fp8, test in ((False, test_tiles_gpu.test_forward_on_both_sides_of_the_key_split_rule),
                      (True, test_tiles_gpu.test_fp8_forward_on_both_sides_of_the_key_split_rule)):
        for d, causal, N, most in _parameters(test, "d", "causal", "N", "most"):
            assert key_split(fp8, most, N, d, causal) and not key_split(fp8, most + 16, N, d, causal), (fp8, d, causal, N, most)


ONE_LAUNCH = {"one32", "rows behind", "rows ahead"}


def test_tests_of_the_backward_rule_lie_on_both_sides_of_it(backward_form):
    def sides(test, *names):
        for d, causal, N, group, most in _parameters(test, *names):
            yield tuple(backward_form(kv * group, kv, N, d, causal) for kv in (most, most + 1)), (d, causal, N, group, most)

    five = "d", "causal", "N", "group", "most"
    for got, case in sides(test_tiles_gpu.test_backward_on_both_sides_of_the_key_split_rule, *five):
        assert got == ("keys32", "large"), (got, case)
    orders = set()
    for got, case in sides(test_tiles_gpu.test_backward_on_both_sides_of_the_rule_of_128_queries, *five):
        assert got[0] == "one32" and got[1].startswith("rows"), (got, case)
        orders.add((case[0], case[1], got[1]))
    assert orders == {(d, c, order) for d in (64, 128) for c in (False, True) for order in ("rows ahead", "rows behind")}
    beyond = set()
    for got, case in sides(test_tiles_gpu.test_backward_both_passes_in_one_launch, *five):
        assert got[0] in ONE_LAUNCH and got[1] not in ONE_LAUNCH, (got, case)
        beyond.add((case[0], case[1], got[1]))
    assert beyond == {(d, c, form) for d in (64, 128) for c in (False, True) for form in ("large", "keys32")}
    for d, causal, N, most in _parameters(test_tiles_gpu.test_backward_on_both_sides_of_the_one_launch_rule, "d", "causal", "N", "most"):
        assert backward_form(most, most, N, d, causal) in ONE_LAUNCH and backward_form(most + 1, most + 1, N, d, causal) not in ONE_LAUNCH, (d, causal, N, most)


def test_tests_of_a_backward_form_take_it(backward_form, own_row_sums):
    for d, N, H in _parameters(test_tiles_gpu.test_backward_shared_score_tiles, "d", "N", "H"):
        if d == 128:
            assert {backward_form(H, H // 2, N, d, c) for c in (False, True)} == {"large"}, (d, N, H)
    for d, N in _parameters(test_tiles_gpu.test_backward_four_wave_query_tiles, "d", "N"):
        assert {backward_form(400, 200, N, d, c) for c in (False, True)} == {"large"}, (d, N)
    for d, causal, N in _parameters(test_tiles_gpu.test_backward_query_tile_rule_edges, "d", "causal", "N"):
        assert backward_form(32, 32, N, d, causal) == "large", (d, causal, N)
    for d, causal, N, group, H_kv in _parameters(test_tiles_gpu.test_backward_32_key_workgroups_by_themselves, "d", "causal", "N", "group", "H_kv"):
        assert backward_form(H_kv * group, H_kv, N, d, causal) == "keys32", (d, causal, N, group, H_kv)
    rows = [(d, causal, backward_form(H, H_kv, N, d, causal), own_row_sums(H, H_kv, N, d)) for d, causal, N, H, H_kv in
            _parameters(test_tiles_gpu.test_backward_128_query_workgroups_beside_key_blocks, "d", "causal", "N", "H", "H_kv")]
    assert {r[2] for r in rows} == {"rows behind", "rows ahead"} and {r[3] for r in rows} == {False, True}
    assert {r[:3] for r in rows} == {(d, c, order) for d in (64, 128) for c in (False, True) for order in ("rows ahead", "rows behind")}
    for H, H_kv, N in _parameters(test_tiles_gpu.test_backward_query_split_for_few_key_blocks, "H", "H_kv", "N"):
        assert {backward_form(H, H_kv, N, d, c) for d in (64, 128) for c in (False, True)} <= ONE_LAUNCH, (H, H_kv, N)


def test_tests_of_row_sums_lie_on_both_sides_of_their_rule(backward_form, own_row_sums):
    cases = _parameters(test_tiles_gpu.test_backward_row_sums_inside_the_one_launch, "d", "N", "H", "H_kv")
    for d, N, H, H_kv in cases:
        assert {backward_form(H, H_kv, N, d, c) for c in (False, True)} <= ONE_LAUNCH, (d, N, H, H_kv)
        if N > 3:  # in pairs: one row more, or one head
            inside = (d, N, H, H_kv) in cases and own_row_sums(H, H_kv, N, d)
            assert (d, N + 1, H, H_kv) in cases or (d, N, H + 1, H_kv + 1) in cases or not inside, (d, N, H, H_kv)
    assert {(d, own_row_sums(H, H_kv, N, d)) for d, N, H, H_kv in cases} == {(d, own) for d in (64, 128) for own in (False, True)}


def test_outputs_over_inputs_are_tested_in_every_backward_form(backward_form, own_row_sums):
    seen = {(d, form, own_row_sums(H, H_kv, N, d) if form in ONE_LAUNCH else N > 1280)
            for d, H, H_kv, N, causal in test_tiles_gpu._FORMS if d < 256 for form in [backward_form(H, H_kv, N, d, causal)]}
    want = {("one32", False), ("one32", True), ("rows ahead", False), ("rows ahead", True), ("rows behind", False), ("keys32", False), ("large", False), ("large", True)}
    assert seen == {(d, *w) for d in (64, 128) for w in want}


@pytest.mark.parametrize("d", [64, 128])
def test_backward_rule_at_the_ends_of_its_range(backward_form, d):
    # one row, the longest head, the most rows a call may have: large wherever the estimates were not compared with times
    longest = 0x7ff00000 // (4 * d)
    for causal in (False, True):
        assert backward_form(1, 1, 1, d, causal) == "one32"
        for heads, kv_heads, N in ((1, 1, longest), (256, 1, longest), ((1 << 31) - 1, (1 << 31) - 1, 1), (1 << 26, 1, 31), (1 << 24, 1 << 20, 100)):
            assert backward_form(heads, kv_heads, N, d, causal) == "large", (heads, kv_heads, N, causal)

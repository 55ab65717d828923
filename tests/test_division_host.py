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
def key_split(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    lib = str(tmp_path_factory.mktemp("division") / "query.so")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "division", "query.cpp"), "-o", lib],
                   check=True, stderr=subprocess.DEVNULL)
    fn = ctypes.CDLL(lib).key_split
    fn.argtypes = [ctypes.c_int, ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return lambda fp8, heads, N, d, causal: bool(fn(int(fp8), heads, N, d, int(causal)))


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

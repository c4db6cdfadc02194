"""The rules that choose a call's kernels by its sizes, and the sizes that they rest
on: the expressions of the internal header, compiled and evaluated on the CPU."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


@pytest.fixture(scope="module")
def evaluate(tmp_path_factory):
    """evaluate([C++ integer expressions]) -> their values."""
    where = tmp_path_factory.mktemp("rules")

    def run(exprs):
        src, exe = str(where / "rules.cpp"), str(where / "rules")
        lines = "\n".join(f'std::printf("%lld\\n", (long long)({e}));' for e in exprs)
        with open(src, "w") as f:
            f.write('#include <cstdio>\n#include "hg_internal.hpp"\nusing namespace hg;\n'
                    f"int main() {{\n{lines}\n}}\n")
        cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__=1", "-I",
               os.path.join(ROOT, "include"), "-I",
               os.path.join(ROOT, "paper_2112_15345_amd", "csrc"), "-isystem", "/opt/rocm/include",
               src, "-o", exe]
        res = subprocess.run(cmd, capture_output=True, text=True)
        assert res.returncode == 0, res.stderr
        out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
        return [int(x) for x in out.split()]

    return run


def test_tiles_of_sparse_types_have_a_pair_table(evaluate):
    """A tile of the layer-wise edge passes whose pairs have one in-edge each, and
    as many empty pairs between them, still has the table of its positions' pairs."""
    pairs, tile = evaluate(["kTilePairs", "kEdgeTile"])
    assert pairs >= 2 * tile


def test_large_bins_are_shared_by_blocks(evaluate):
    """A bin of any number of records is summed in parts of at most 32768 records, one
    to a block, and the bounds on the parts and on the bins in parts hold."""
    sizes = [1, 32767, 32768, 32769, 65536, 65537, 1 << 20, (1 << 31) - 1]
    part, *n = evaluate(["kBinPart"] + [f"bin_parts({r})" for r in sizes])
    for r, k in zip(sizes, n):
        assert (k == 0 and r <= part) or (k >= 2 and (k - 1) * part < r <= k * part)
    # bins that make the most of n in-edges: all just over a part
    for n_bins in (1, 3, 100):
        total = n_bins * (part + 1)
        large, parts = evaluate([f"most_large_bins({total}, {n_bins})",
                                 f"most_bin_parts({total})"])
        assert large == n_bins and parts >= 2 * n_bins
    # many in-edges from a type of few bins: no more sums than it has bins
    assert evaluate([f"most_large_bins({(1 << 31) - 1}, {b})" for b in (2, 8192)]) == [2, 8192]


def test_active_pairs_of_sparse_masks_only(evaluate):
    """A hop lists its active pairs where they are few of many: never with half of
    them active (going through every pair is faster at all sizes), and from some size
    on with a few per cent, later with more active ones or more edge types."""
    sizes = [1 << k for k in range(10, 31)]

    def first(share, words):
        pays = evaluate([f"active_pairs_pay({p}, {int(p * share)}, {words})" for p in sizes])
        assert pays == sorted(pays)  # from some size on
        return sizes[pays.index(1)] if 1 in pays else None

    assert first(0.5, 1) is None and first(1.0, 7) is None
    assert 1 << 18 < first(0.03, 1) <= first(0.03, 7) <= 1 << 20
    assert first(0.03, 2) <= first(0.2, 2) <= first(0.3, 2) <= 1 << 21


def test_pair_bits_grid(evaluate):
    """The pass over the node types of every copy of a bundle (here up to 32 of more
    than 2048 types) launches a grid that the device takes, with few idle blocks, and
    enough of them for one type's frontier."""
    cases = [(f, t) for t in (1, 4, 1024, 1025, 67_200, 1_000_000)
             for f in (0, 1, 193, 100_000, 1 << 31)]
    got = evaluate([f"pair_bits_grid({f}, {t}).{c}" for f, t in cases for c in "xy"])
    for (front, types), x, y in zip(cases, got[::2], got[1::2]):
        assert 1 <= y <= min(types, 65_535) and 1 <= x <= 4096 and x * y <= 1 << 16
        assert y == types or types > 1024
        if types <= 4:
            assert x == min(4096, (front + 64 + 255) // 256)


@pytest.fixture(scope="module")
def compile_sampler(tmp_path_factory):
    """compile_sampler(*options) -> the sampler's device code as the compiler's text."""
    from paper_2112_15345_amd import build
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")

    def run(*options):
        out = str(tmp_path_factory.mktemp("sampler") / "sample.txt")
        cmd = [hipcc, "-x", "hip", *build.COMMON, "--offload-device-only", "-S", *options,
               os.path.join(build.CSRC, "hg_sample.hip"), "-o", out]
        res = subprocess.run(cmd, capture_output=True, text=True)
        assert res.returncode == 0, res.stderr
        return open(out).read()

    return run


def test_candidate_threshold_has_one_value(compile_sampler):
    """The sampler computes a hub's candidate threshold in several places, which must
    agree to the bit: the compiler may contract or reorder none of its operations (a
    multiply and an add fused in one place and not in another would differ)."""
    ops = re.findall(r"= (f(?:add|sub|mul|div)\b[^%]*)float", compile_sampler("-emit-llvm"))
    assert ops  # its operations are there
    assert not [x for x in ops if x.split()[1:]], "arithmetic with fast-math flags"


def test_counting_pass_leaves_room_for_two_blocks(compile_sampler):
    """Every variant of the counting pass, as built, and the largest table of edge
    types that it is launched with take at most half of a CU's 160 KiB of LDS."""
    code = compile_sampler()
    limit = int(re.search(r"kCountMaxEtypes = (\d+)", open(os.path.join(
        ROOT, "paper_2112_15345_amd", "csrc", "hg_sample.hip")).read()).group(1))
    own = [int(n) for n in re.findall(
        r"\.amdhsa_kernel \S*k_count_scan\S*\n\s*\.amdhsa_group_segment_fixed_size (\d+)", code)]
    assert len(own) == 6 and max(own) >= 16 * 1024  # the striped ones among them
    assert max(own) + 36 * limit + 8 <= 160 * 1024 // 2

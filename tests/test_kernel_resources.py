"""Registers, scratch memory and LDS of the kernels in the built library, from the notes of its code objects: what decides how many
wavefronts share a SIMD (512 registers, eight wavefronts) and how many workgroups a compute unit (160 KiB of LDS)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2102_08124_amd import build

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 code objects of a library: each translation unit embeds a bundle."""
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in name and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """kernel (template arguments, without those of its table) -> list of {vgpr, scratch, lds, threads}"""
    readelf = os.path.join(LLVM, "llvm-readelf")
    if not os.path.exists(readelf) or not shutil.which("c++filt"):
        pytest.skip("no llvm-readelf or c++filt")
    if not os.path.exists(build.LIB):
        build.build()
    folder, found = tmp_path_factory.mktemp("objects"), []
    for k, code in enumerate(_code_objects(open(build.LIB, "rb").read())):
        path = folder / ("%d.co" % k)
        path.write_bytes(code)
        notes = subprocess.run([readelf, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
        for entry in re.split(r"\n\s*- \.agpr_count:", notes)[1:]:
            field = lambda name: int(re.search(r"\.%s:\s+(\d+)" % name, entry).group(1))
            found.append((re.search(r"\.symbol:\s+(\S+)\.kd", entry).group(1),
                          dict(vgpr=field("vgpr_count"), scratch=field("private_segment_fixed_size"), lds=field("group_segment_fixed_size"),
                               threads=field("max_flat_workgroup_size"))))
    names = subprocess.run(["c++filt"], input="\n".join(n for n, _ in found), check=True, capture_output=True, text=True).stdout.split("\n")
    out = {}
    for name, (_, use) in zip(names, found):
        name = re.sub(r"\(.*|tmask::|^void ", "", name)
        out.setdefault(re.sub(r"(, )?(Few)?(Batch|Pack)ArgsOf<\d+> ?|\s+(?=>)", "", name), []).append(use)
    assert len(out) > 100
    return out


def _wavefronts(use):
    """of a SIMD, by registers (allocated in eights)"""
    return min(8, 512 // (-(-use["vgpr"] // 8) * 8))


@pytest.mark.parametrize("name,waves", [("cw_exact_kernel<%d, 8, %d>", 6), ("cw_score_kernel<%d, 32, 1>", 7)])
@pytest.mark.parametrize("dt", [0, 1])
def test_column_per_lane_kernels_hold_nothing_for_their_end(kernels, name, waves, dt):
    """Where a workgroup's sum goes is read behind the loop over tiles."""
    for fmt in (0, 1):
        use, = kernels[name % ((dt, fmt) if name.count("%") == 2 else dt)]
        assert _wavefronts(use) >= waves and use["scratch"] == 0, use


@pytest.mark.parametrize("fmt", [0, 1])
def test_16_of_32_by_rows_has_eight_workgroups_on_a_compute_unit(kernels, fmt):
    use, = kernels["cw_mask32_bf16_kernel<%d>" % fmt]
    assert use["threads"] == 256 and _wavefronts(use) == 8 and 160 * 1024 // use["lds"] >= 8, use


@pytest.mark.parametrize("m,waves", [(8, 5), (16, 3)])
def test_the_exact_kernels_keep_next_to_nothing_in_scratch_memory(kernels, m, waves):
    """At most four values of a lane at M = 8, two at M = 16 (and 4 bytes); their workgroups are four wavefronts."""
    for dt in (0, 1):
        for fmt in (0, 1):
            for general in ("false", "true"):
                use, = kernels["exact_balanced_kernel<%d, %d, %d, %s>" % (dt, m, fmt, general)]
                none = m == 8 and (dt, fmt, general) != (1, 1, "true")
                assert _wavefronts(use) == waves and use["scratch"] <= (0 if none else 20 if m == 8 else 12), (dt, fmt, general, use)


def test_column_per_lane_kernels_of_small_calls_hold_all_in_registers(kernels):
    uses = [(name, use) for name, found in kernels.items() if re.match("exact_spread|approx_spread16", name) for use in found]
    assert len(uses) == 48
    for name, use in uses:
        assert use["scratch"] == 0, (name, use)
        if name.startswith("exact_spread_kernel<") and ", 16," in name:
            assert min(_wavefronts(use), 160 * 1024 // use["lds"]) >= 5, (name, use)     # of 256 threads: up to where they are chosen


@pytest.mark.parametrize("name", ["approx_sel_f32_kernel<16, %d, true>", "approx_dense_kernel<0, 16, %d, 0>"])
@pytest.mark.parametrize("fmt", [0, 1])
def test_any_n_at_m16_fits_four_wavefronts(kernels, name, fmt):
    """Algorithm 1 on fp32: the weights are held once, magnitudes are taken where they are needed."""
    use, = kernels[name % fmt]
    assert _wavefronts(use) == 4 and use["scratch"] == 0, use


@pytest.mark.parametrize("dt", [0, 1, 2])
@pytest.mark.parametrize("fmt", [0, 1])
def test_scores_at_m4_leave_room_for_eight_wavefronts(kernels, dt, fmt):
    """They are bound by what they read; records that are added up in the launch must not cost them a wavefront."""
    uses = kernels["score_kernel<%d, 4, %d>" % (dt, fmt)]
    assert len(uses) == 2                                      # the two sizes of the table
    for use in uses:
        assert _wavefronts(use) == 8 and use["scratch"] == 0, use


def test_no_form_of_algorithm_1_that_nothing_takes(kernels):
    assert not [name for name in kernels if re.match(r"mask_kernel<0, \d, (8|16),", name)]


def test_a_compute_unit_has_three_places_for_each_kernel_that_waits(kernels):
    """What the number of workgroups that may wait in a launch is reckoned with."""
    waits = re.compile(r"mask_kernel<|approx24|approx_sel|approx_spread16_kernel<\d, false|exact24|exact_balanced|exact_spread|score_kernel<|approx_pack24|pack48_\w+<.*true|cw_mask|cw_exact|cw_score")
    seen = wide = 0
    for name, uses in kernels.items():
        if not waits.match(name):
            continue
        for use in uses:
            lds = use["lds"] + (8192 if name.startswith("approx_pack24_kernel<0") else 0)         # reserved at the launch
            places = min(_wavefronts(use) * 4 // (use["threads"] // 64), 160 * 1024 // lds if lds else 32)
            assert places >= 3, (name, use)
            seen += 1
            wide += use["threads"] == 512
    assert seen > 100 and wide == 10              # 512 threads: the optimal masks at M = 8 and Algorithm 1 for bf16 at M = 16, in small calls

"""The rule that gives a retrieval one wave per component (split_plan), asked on
the CPU: on each side of every line it takes the form that was measured faster
there, and the register budgets it counts with are the compiled kernels'."""
import os
import re
import shutil
import subprocess

import pytest

from conftest import ROOT

LLVM = "/opt/rocm/llvm/bin/"
CSRC = os.path.join(ROOT, "paper_2308_11759_amd", "csrc")

# (type, components, waves, box, one wave per component is faster), us for one
# wave for all / one per component measured on whole cubes (boxes: of 300^3 and
# 512^3) with about 540 payload words to a wave and component.  Types: codec 0
# on the high-half routes, codec 0 off them ("wide"), codec 1.
MEASURED = [
    ("f32", 8, 512, 0, True), ("f32", 8, 729, 0, True), ("f32", 8, 858, 0, False),  # 48/31 48/43 48/55
    ("f32", 7, 512, 0, True), ("f32", 7, 858, 0, False),  # 42/31 43/54
    ("f32", 6, 512, 0, True), ("f32", 6, 729, 0, False), ("f32", 6, 1000, 0, False),  # 37/30 37/41 37/53
    ("f32", 5, 512, 0, True), ("f32", 5, 729, 0, False), ("f32", 5, 1000, 0, False),  # 32/29 32/41 33/53
    ("f32", 4, 729, 0, True), ("f32", 4, 858, 0, False), ("f32", 4, 1728, 0, False),  # 28/22 29/31 38/45
    ("f32", 3, 1000, 0, True), ("f32", 3, 1331, 0, False),  # 24.8/24.3 30/39
    ("f32", 2, 216, 0, True), ("f32", 2, 275, 0, False), ("f32", 2, 1728, 0, False),  # 19.2/18.6 20.0/20.7 26/35
    ("f32", 8, 648, 1, True), ("f32", 6, 648, 1, True), ("f32", 5, 648, 1, False),  # 63/47 50/46 44.7/45.4
    ("f32", 5, 1058, 1, False), ("f32", 6, 1152, 1, False), ("f32", 8, 1152, 1, False),  # 46/69 54/68 69/72
    ("f32", 4, 1152, 1, True), ("f32", 4, 1568, 1, False),  # 43/35 41/47
    ("f32", 3, 800, 1, True), ("f32", 3, 1058, 1, False),  # 35/26 35.1/35.8
    ("f32", 2, 1352, 1, True), ("f32", 2, 1568, 1, False),  # 29/28 29/37
    ("f32wide", 8, 729, 0, True), ("f32wide", 6, 729, 0, True), ("f32wide", 5, 729, 0, False),  # 55/47 50/45 43/45
    ("f32wide", 4, 1000, 0, True), ("f32wide", 2, 729, 0, True), ("f32wide", 2, 858, 0, False),  # 35/32 21/19 21.5/22.5
    ("f32pred", 8, 729, 0, True), ("f32pred", 6, 729, 0, True), ("f32pred", 5, 729, 0, False),  # 42/34 34/32 29/32
    ("f32pred", 4, 1000, 0, True), ("f32pred", 2, 216, 0, True), ("f32pred", 2, 343, 0, False),  # 26/23 15.2/14.7 15.5/16.2
    ("f64", 8, 512, 0, True), ("f64", 8, 615, 0, False), ("f64", 7, 512, 0, True),  # 48/41 48/58 43/40
    ("f64", 5, 216, 0, True), ("f64", 5, 275, 0, False),  # 32/21 33/37
    ("f64", 4, 512, 0, True), ("f64", 4, 615, 0, False), ("f64", 3, 512, 0, True), ("f64", 3, 615, 0, False),
    # 30/23 31/36 26/23 27/34
    ("f64", 2, 1000, 0, True), ("f64", 2, 1331, 0, False),  # 26/23 29/38
    ("f64wide", 4, 245, 0, True), ("f64wide", 3, 275, 0, False), ("f64wide", 6, 245, 0, True),  # 37/22 29/35 52/40
    ("f64wide", 6, 275, 0, False), ("f64wide", 2, 512, 0, True), ("f64wide", 2, 615, 0, False),  # 53/70 23/22 24/36
    # more components than a launch takes
    ("f32", 9, 343, 0, True), ("f32", 10, 245, 0, True), ("f32", 10, 343, 0, False),  # 44/41 46/31 48/50
    ("f32", 12, 512, 0, True), ("f32", 12, 729, 0, False), ("f32", 16, 729, 0, False),  # 56/53 56/76 75/82
    ("f32pred", 10, 343, 0, True), ("f32pred", 16, 729, 0, True), ("f32pred", 12, 729, 0, False),  # 48/44 75/69 57/65
    ("f64", 12, 245, 0, True), ("f64", 12, 343, 0, False), ("f64", 16, 343, 0, True),  # 67/41 64/72 81/78
    ("f64pred", 4, 245, 0, True), ("f64pred", 3, 275, 0, False), ("f64pred", 8, 245, 0, True),  # 28/19 23/29 47/35
]


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("split") / "split_rule")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "native", "split_rule.cpp"), "-o", exe], check=True)

    def run(lines):
        text = "".join("%d %d %d %d %d %d %d %d %d\n" % l for l in lines)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in l.split()) for l in out.splitlines()]

    return run


def line(kind, k, waves, box, i0=0, span=540):
    """Flags: 1 a block outside the 16-bit routes, 2 outside the 32-bit one, 4 raw."""
    first = 7 if kind == "f64wide" else 1
    rest = 0 if kind in ("f32", "f64") else 1
    return (1 if kind.startswith("f32") else 2, int(kind.endswith("pred")), first, rest, span, i0, k, waves, box)


def test_the_faster_form_at_every_line(ask):
    got = ask([line(t, n, w, box) for t, n, w, box, _ in MEASURED])
    wrong = [m for m, g in zip(MEASURED, got) if (g[0] == 1) != m[4]]
    assert not wrong


def test_every_plan_fits_its_launch(ask):
    """Components per launch, LDS and the launches' cover, over the whole range."""
    for kind in ("f32", "f32wide", "f32pred", "f64", "f64wide", "f64pred"):
        most = 4 if kind in ("f64wide", "f64pred") else 8
        for k in range(1, 33):
            for i0 in range(0, k):
                lines = [line(kind, k, w, box, i0, span) for w in (1, 255, 257, 2000) for box in (0, 1)
                         for span in (1, 540, 1700, 9000, 20000)]
                for l, g in zip(lines, ask(lines)):
                    if g[0]:
                        n = g[1] - i0
                        cap = (l[4] + 63) // 64 * 64
                        assert 2 <= n <= most and g[1] <= k
                        assert max(n * (cap + 3) * 4, n * 4096) == g[2] <= 65536 - 512


def test_registers_hold_the_waves_the_rule_counts(tmp_path):
    """512 registers per SIMD lane and four SIMDs: twelve float32 waves per CU
    need at most 168 each, eight float64 ones on the high-half routes 256."""
    lib = os.path.join(ROOT, "paper_2308_11759_amd", "libpmc.so")
    if not (os.path.exists(lib) and os.path.exists(LLVM + "llvm-objdump")):
        pytest.skip("needs the built library and ROCm's LLVM tools")
    copy = shutil.copy(lib, tmp_path)
    subprocess.run([LLVM + "llvm-objdump", "--offloading", copy], check=True, capture_output=True, cwd=tmp_path)
    seen = 0
    for f in sorted(os.listdir(tmp_path)):
        if "gfx950" not in f:
            continue
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", os.path.join(tmp_path, f)], check=True,
                               capture_output=True, text=True).stdout
        for kernel in notes.split("  - .agpr_count")[1:]:
            m = re.search(r"\.name:\s+_ZN3pmc14k_decode_splitI([fd])Lb(\d)ELi(\d)ELb(\d)E", kernel)
            if not m:
                continue
            total = int(re.search(r"\.vgpr_count:\s+(\d+)", kernel).group(1))
            spilled = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
            t, hires = m.group(1), m.group(4) == "1"
            assert total <= (168 if t == "f" else 256 if hires else 512), (m.group(0), total)
            assert spilled == 0, (m.group(0), spilled)
            seen += 1
    assert seen == 12

"""What the build refuses: kernels that spill scalar registers where the inline assembly relies on none, softmax slots that would end behind the check of their results."""
import os
import shutil
import subprocess

import pytest

from paper_2602_06072_amd import build


def remarks(*kernels):
    return "".join(f"x.hip:1:1: remark: Function Name: {name} [-Rpass-analysis=kernel-resource-usage]\n"
                   f"x.hip:1:1: remark:     VGPRs Spill: 2 [-Rpass-analysis=kernel-resource-usage]\n"
                   f"x.hip:1:1: remark:     SGPRs Spill: {n} [-Rpass-analysis=kernel-resource-usage]\n" for name, n in kernels)


def test_scalar_spills_are_found():
    assert build.scalar_spills(remarks(("a", 0), ("b", 0))) == []
    assert build.scalar_spills(remarks(("a", 0), ("b", 3))) == [("b", 3)]
    for nothing in ("", "warning: something else\n", "remark: Function Name: a\n"):
        with pytest.raises(RuntimeError):
            build.scalar_spills(nothing)


def test_kernels_with_such_copies_are_checked(monkeypatch, tmp_path):
    """Every source file that includes the body with the copies; and the compiler's remarks are in the form that is read."""
    for src in build.SOURCES:
        text = open(f"{build.CSRC}/{src}").read()
        assert ('#include "prefill_body.hip.h"' in text) == (src in build.NO_SCALAR_SPILLS), src
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    seen = []
    real = build.scalar_spills
    monkeypatch.setattr(build, "scalar_spills", lambda t: seen.append(t) or [("kernel", 1)])
    with pytest.raises(RuntimeError, match="scalar registers spill"):
        build._compile("prefill_pipe.hip")
    assert real(seen[0]) == [] and "prefill_bf16_pair_kernel" in seen[0]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("spare, builds", [(4, True), (3, False)])
def test_softmax_slots_leave_room_for_the_check(tmp_path, spare, builds):
    """With a spare slot less the last pair of head dimension 64 would be combined behind the branch that looks for large probabilities."""
    for name in os.listdir(build.CSRC):
        if name.endswith((".h", ".hip")):
            shutil.copy(os.path.join(build.CSRC, name), tmp_path)
    header = tmp_path / "prefill_body.hip.h"
    text = header.read_text()
    line = "constexpr int SPARE = D == 128 ? 2 * NC : 4;"
    assert line in text
    header.write_text(text.replace(line, line.replace(": 4;", f": {spare};")))
    run = subprocess.run(["hipcc", *build.HIP_FLAGS, "-fsyntax-only", "--offload-device-only", str(tmp_path / "prefill_pipe.hip")],
                         capture_output=True, text=True)
    assert (run.returncode == 0) == builds, run.stderr[-2000:]
    assert builds or "packed and combined before the check" in run.stderr

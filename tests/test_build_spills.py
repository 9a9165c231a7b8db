"""The build refuses kernels that spill scalar registers where the inline assembly relies on none."""
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

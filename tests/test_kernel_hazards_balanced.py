"""The wait-state check of test_kernel_hazards on the balanced launch's kernels:
the same steps inside a loop over pieces, so that a path may lead from one piece's
MFMAs into the next piece's code."""
import re

from test_kernel_hazards import (NEED, _shortest_use, attention_asm)  # noqa: F401 (fixture)


def _balanced_kernels(asm: str):
    for name in sorted(set(re.findall(r"^(_ZN2ca25balanced_attention_kernel\w+):", asm, re.M))):
        at = asm.index(name + ":")
        lines, labels = [], {}
        for raw in asm[at:asm.index(".Lfunc_end", at)].split("\n")[1:]:
            text = raw.split(";")[0].strip()
            m = re.match(r"^(\.LBB\d+_\d+):", text)
            if m:
                labels[m.group(1)] = len(lines)
            elif text and not text.startswith("."):
                lines.append(text)
        yield name, lines, labels


def test_balanced_mfma_results_wait_before_use(attention_asm):  # noqa: F811
    kernels = list(_balanced_kernels(attention_asm))
    # D in {64, 128} x {selected, dense} x V layout in {token-major, transposed}
    assert len(kernels) == 8
    for name, lines, labels in kernels:
        mfma = [k for k, text in enumerate(lines) if text.startswith("v_mfma")]
        assert len(mfma) >= 64, name
        for k in mfma:
            d = _shortest_use(lines, labels, k)
            assert d is None, f"{name}: {lines[k]} is used after {d} wait states (< {NEED})"

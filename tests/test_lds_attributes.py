"""CPU: kernels that take more than the default LDS opt in once per variant, through one helper that both the
launch and the preparation before a graph capture call, so that no launch inside a capture is the first."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1412_2293_amd", "csrc")


def functions_calling(text, name):
    """Names of the top-level functions whose bodies call `name`."""
    out, current = [], None
    for line in text.splitlines():
        m = re.match(r"^(?:static |template\S* )*(?:hipError_t|int|bool|size_t|void) (\w+)\(", line)
        if m:
            current = m.group(1)
        if re.search(r"\b%s\b *[(<]" % name, line) and not (m and m.group(1) == name):
            out.append(current)
    return out


@pytest.mark.parametrize("source,helper,users", [
    ("fused_kernel.h", "fused_attr_one", {"launch_t", "fused_attributes"}),
    ("state.hip", "state_attr_one", {"state_launch_t", "state_prepare_attributes"}),
])
def test_lds_opt_in_is_shared_by_launch_and_preparation(source, helper, users):
    text = open(os.path.join(CSRC, source)).read()
    assert set(functions_calling(text, "hipFuncSetAttribute")) == {helper}
    assert users <= set(functions_calling(text, helper))
    body = text[text.index(f"static hipError_t {helper}()"):]
    assert "static const hipError_t attr" in body[:body.index("\n}\n")]

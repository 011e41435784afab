"""Barriers of the kernels that avoid the full workgroup fence, read from the
sources: a kernel whose waves store to LDS publishes it by barrier_lds (each
wave waits for its own stores first); barrier_nofence alone is for kernels
whose LDS is written by direct global->LDS loads only.  No run can show a
missing wait dependably, so the call sites are checked instead."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_25422_amd", "csrc")


def kernel_body(source, name):
    """Text of kernel `name`, from its name to the brace that closes it."""
    text = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, source)).read())
    m = re.search(r"__global__[^;{]*\b" + name + r"\s*\(", text)
    assert m, name
    i = text.index("{", m.end())
    depth, j = 1, i + 1
    while depth:
        depth += {"{": 1, "}": -1}.get(text[j], 0)
        j += 1
    return text[i:j]


@pytest.mark.parametrize("source,name", [("mlp.hip", "mlp_score_kernel"),
                                         ("attn.hip", "attn_sparse_kernel")])
def test_kernels_that_store_to_lds_wait_for_their_stores(source, name):
    body = kernel_body(source, name)
    assert "barrier_lds()" in body
    assert "barrier_nofence()" not in body and "builtin_amdgcn_s_barrier" not in body


@pytest.mark.parametrize("name", ["proj_gemm_kernel", "proj_wide_kernel"])
def test_the_plain_barrier_only_publishes_direct_loads(name):
    """The projection tiles' one LDS array is filled by lds_dma16 alone."""
    body = kernel_body("proj.hip", name)
    assert "barrier_nofence()" in body
    assert re.findall(r"__shared__[^;]*\b(\w+)\[", body) == ["Ar"]
    assert not re.search(r"\b(Ar|At)\b[^;=]*[^=!<>]=[^=]", body.replace("const bf16_t* At = Ar", ""))

"""Promises that kernel signatures make to the compiler (no GPU)."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_24504_amd", "csrc")


def test_published_scalars_are_not_restrict():
    """The Gram-Schmidt kernels store coefficients (h, hout) into the scalar block that the same
    launch publishes through pub.src: a restrict pointer would promise that no other reads them."""
    with open(os.path.join(CSRC, "la.hip")) as fh:
        text = fh.read()
    for kernel, arg in (("update_kernel", "h"), ("update2_kernel", "hout")):
        params = re.search(r"\n" + kernel + r"\((.*?)\)\n\{", text, re.S)[1]
        assert "Publish pub" in params
        decl, = [q.strip() for q in params.split(",") if re.search(r"\b" + arg + r"$", q.strip())]
        assert "const" not in decl and "__restrict__" not in decl, decl

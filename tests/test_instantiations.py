"""A body's arithmetic is the same alone and in a batch: the marker kernels exist in a form for a lone
body and a form for several, and the compiler may fuse a product and a sum in one form and not in the
other.  That shows in one bit of one value in millions, which no run of reasonable length meets, so the
generated code is compared: both forms of a kernel hold the same numbers of floating-point operations."""
import collections
import os
import re
import subprocess

KERNEL = re.compile(r"^_ZN4lbib\d+(k_[a-z_]+)ILb([01])E(\w*?)Evi?NS_5PoolsE?\w*:")
OPS = {"fma": "fused", "fmac": "fused", "fmaak": "fused", "fmamk": "fused", "mul": "product",
       "add": "sum", "sub": "sum", "subrev": "sum", "rcp": "rcp", "rsq": "rsq", "sqrt": "sqrt", "exp": "exp"}


def test_lone_and_batched_marker_kernels_do_the_same_arithmetic(tmp_path):
    from paper_2207_06029_amd import build as B
    asm = str(tmp_path / "ib.s")
    r = subprocess.run([B.HIPCC, *B.FLAGS, "--offload-device-only", "-S", os.path.join(B.CSRC, "lbib_ib.hip"), "-o", asm],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    forms, ops = collections.defaultdict(dict), None
    for line in open(asm):
        if line.startswith("_Z"):
            m = KERNEL.match(line)
            ops = forms[m.group(1), m.group(3)].setdefault(m.group(2), collections.Counter()) if m else None
        elif ops is not None:
            m = re.match(r"\s+v_([a-z]+)_(f32|f64)", line)
            if m and m.group(1) in OPS:
                ops[OPS[m.group(1)], m.group(2)] += 1
    assert {k for k, _ in forms} == {"k_centroids", "k_triangles", "k_vertices"}
    for key, form in forms.items():
        assert set(form) == {"0", "1"} and form["1"]["fused", "f64"] > 0, key
        assert form["0"] == form["1"], key

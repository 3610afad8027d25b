"""A body's arithmetic is the same alone and in a batch: the marker kernels exist in a form for a lone
body and a form for several, and the compiler may fuse a product and a sum in one form and not in the
other.  That shows in one bit of one value in millions, which no run of reasonable length meets, so the
generated code is compared: both forms of a kernel hold the same numbers of floating-point operations.
The one-lattice sweeps, the hot kernels of their storage forms, keep their values in registers."""
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


def _kernels(so):
    """Metadata of every kernel in the built library's device code objects."""
    data = open(so, "rb").read()
    out, at = {}, data.find(b"\x7fELF", 1)
    while at > 0:
        nxt = data.find(b"\x7fELF", at + 1)
        obj = data[at:nxt if nxt > 0 else len(data)]
        r = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", "-"], input=obj, capture_output=True)
        for block in re.split(r"\n\s+- \.", r.stdout.decode())[1:]:
            m = re.search(r"\.symbol:\s+(\S+)\.kd", block)
            if m:
                out[m.group(1)] = {k: int(v) for k, v in re.findall(r"(\w+):\s+(\d+)\n", block)}
        at = nxt
    return out


def test_sweeps_of_one_lattice_spill_no_vector_register():
    from paper_2207_06029_amd import build as B
    sweeps = {k: v for k, v in _kernels(B.SO).items() if re.match(r"_ZN4lbib7k_sweepI\w+Lb1ELi1ELb[01]ELb1E", k)}
    assert len(sweeps) == 6   # three storage forms, 32- and 64-bit offsets
    for k, v in sweeps.items():
        assert v["vgpr_spill_count"] == 0 and v["private_segment_fixed_size"] == 0, k

"""CPU: the export and import kernels (csrc/kv_transfer.h), compiled for gfx950, store 8 elements per instruction: 16 bytes of
bfloat16, 8 of codes, and nothing narrower."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    from paper_2509_24381_amd.build import HIPCC_FLAGS
    src = tmp_path_factory.mktemp("isa") / "kernels.hip"
    kernels = ["kv_%s_kernel<%d, %s, %s>" % (k, d, t, c) for k in ("export", "import") for d in (64, 128)
               for t, c in (("bf16", "bf16"), ("uint8_t", "bf16"), ("uint8_t", "uint8_t"))]
    args = {"export": "%s* k, %s* v", "import": "const %s* k, const %s* v"}
    text = '#include "kv_transfer.h"\n'
    for name in kernels:
        c = name.rstrip(">").split(", ")[2]
        text += "template __global__ void %s(ReqDesc, Fp8CacheDesc, KVPageWindow, int, %s, int, int, int);\n" % (
            name, args[name[3:9]] % (c, c))
    src.write_text(text)
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    out = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-I", os.path.join(ROOT, "paper_2509_24381_amd", "csrc"),
                          "--cuda-device-only", "-S", str(src), "-o", "-"], capture_output=True, text=True, check=True).stdout
    return dict(re.findall(r"^(_Z\w*kv_(?:ex|im)port_kernel\w*):(.*?)^\.Lfunc_end", out, re.M | re.S))


@pytest.mark.parametrize("kind", ["export", "import"])
def test_stores_are_eight_elements_wide(assembly, kind):
    bodies = {k: v for k, v in assembly.items() if kind in k}
    assert len(bodies) == 6
    for name, body in bodies.items():
        stores = set(re.findall(r"global_store_(\w+)", body))
        cache, canonical = re.search(r"ILi\d+E(h|DF16b)(h|DF16b)E", name).groups()   # mangled element types
        codes = (canonical if kind == "export" else cache) == "h"
        assert stores == ({"dwordx2"} if codes else {"dwordx4"}), f"{name}: {sorted(stores)}"

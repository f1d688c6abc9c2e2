"""What the compiler gave the kernels of the built library, from the metadata
of its own code objects: no pair pass, in any variant, keeps anything in
scratch memory."""
import os
import re
import struct
import subprocess

import pytest

wc = pytest.importorskip("paper_2609_05494_amd")
from paper_2609_05494_amd import build as hb  # noqa: E402

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(path):
    blob = open(path, "rb").read()
    for m in re.finditer(MAGIC, blob):
        at = m.end()
        (n,) = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + length].decode()
            at += 24 + length
            if "gfx950" in name and size:
                yield blob[m.start() + off:m.start() + off + size]


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: bytes of scratch per lane}"""
    if not os.path.exists(wc.LIB_PATH):
        hb.build()
    out = {}
    for k, co in enumerate(_code_objects(wc.LIB_PATH)):
        p = tmp_path_factory.mktemp("co") / f"{k}.co"
        p.write_bytes(co)
        text = subprocess.run([READELF, "--notes", str(p)], capture_output=True, text=True, check=True).stdout
        names = re.findall(r"^\s+\.name:\s+(_Z\w+)$", text, re.M)
        scratch = re.findall(r"^\s+\.private_segment_fixed_size:\s+(\d+)$", text, re.M)
        assert len(names) == len(scratch)
        out.update(zip(names, map(int, scratch)))
    return out


def test_pair_passes_use_no_scratch(kernels):
    pair = {k: v for k, v in kernels.items() if "k_pair" in k or "k_dens" in k}
    assert len(pair) > 40
    assert not {k: v for k, v in pair.items() if v}

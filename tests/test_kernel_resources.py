"""What the built library's kernels take of a CU, as the compiler wrote it into the code objects' notes: kernels
whose arrays are meant to stay in registers use no LDS or scratch for them."""
import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    from paper_2209_03526_amd import build
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    data = open(build.LIB, "rb").read()
    found, at = {}, data.find(MAGIC)
    while at >= 0:                                            # a bundle for each source file
        count, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in name and size:
                co = str(tmp_path_factory.mktemp("co") / "k.co")
                open(co, "wb").write(data[at + off:at + off + size])
                notes = subprocess.run([READELF, "--notes", co], capture_output=True, text=True, check=True).stdout
                for block in notes.split("  - .agpr_count")[1:]:
                    get = lambda key: re.search(r"\." + key + r":\s+(\S+)", block)[1]  # noqa: E731
                    found[get("symbol")] = (int(get("group_segment_fixed_size")), int(get("private_segment_fixed_size")))
        at = data.find(MAGIC, at + 1)
    assert len(found) > 20
    return found


@pytest.mark.parametrize("kernel", ["k_reshare_calls", "k_csr_select", "k_compact", "k_group_table", "k_rss"])
def test_no_scratch(kernels, kernel):
    mine = {k: v for k, v in kernels.items() if kernel in k}
    assert mine and all(v[1] == 0 for v in mine.values()), mine


def test_the_batched_reshare_needs_no_lds(kernels):
    mine = [v for k, v in kernels.items() if "k_reshare_calls" in k]
    assert mine and all(v[0] == 0 for v in mine)

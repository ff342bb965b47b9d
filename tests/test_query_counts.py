"""The queries' loads through the scalar cache tell the compiler that nothing
writes at the address while the kernel runs.  A kernel that clears the block
counts it has read therefore loads them as ordinary memory, from a pointer
that is not to const: no device source casts constness away, and every
function that stores to the counts reads them through block_count."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1705_03750_amd", "csrc")


def device_source(name):
    with open(os.path.join(CSRC, name)) as f:
        return re.sub(r"//[^\n]*", "", f.read())


def test_no_store_to_constant_memory():
    for name in ("vp_kernels.hpp", "vp_batch.hpp", "vp4_kernels.hpp"):
        assert "const_cast" not in device_source(name), name


def test_cleared_counts_are_ordinary_loads():
    src = device_source("vp_kernels.hpp")
    for fn in ("recon_tile", "remap_tile"):
        body = src[src.index(f"void {fn}("):]
        body = body[:body.index("\n}\n")]
        assert re.search(r"if constexpr \(CLR\) \{\s*if \(lane == 0\) "
                         r"cnt\[b\] = 0;", body), fn
        assert "block_count<CLR>(cnt + b)" in body, fn
        assert "uload(cnt" not in body, fn
    # and that load is through the scalar cache only where nothing is stored
    body = src[src.index("int block_count("):]
    body = body[:body.index("\n}\n")]
    plain, constant = body.split("else")
    assert "if constexpr (CLR)" in plain and "uload" not in plain
    assert "uload" in constant

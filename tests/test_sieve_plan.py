"""Sizes that the threshold-first search plans on the host, compiled for the CPU from
the library's own header and checked over the range that the entry points accept."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1702_08734_amd", "csrc")
SHIM = r"""
#include "sieve_plan.hpp"
extern "C" {
int row_bits() { return mk::kSieveRowBits; }
void chunks(int64_t nqb, int64_t nb, int bn, int64_t* out) {
    mk::plan_sieve_chunks(nqb, nb, bn, &out[0], &out[1]);
}
void batch(int64_t nq, int64_t nb, int keff, int64_t* out) {
    const mk::SievePlan p = mk::plan_sieve(nb, keff);
    out[0] = mk::sieve_batch(nq, nb, keff);
    out[1] = p.cap;
    out[2] = p.sample;
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)],
                   check=True)
    lib = ctypes.CDLL(str(so))
    lib.chunks.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.POINTER(ctypes.c_int64)]
    lib.batch.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.POINTER(ctypes.c_int64)]
    return lib


# a row of a chunk is staged in kSieveRowBits bits, the chunk's length ("past the
# end") too; the chunks cover the rows, none of them empty
@pytest.mark.parametrize("bn", [32, 64, 128])
@pytest.mark.parametrize("nqb", [1, 3, 40, 200, 256, 1000, 4096])
def test_chunks_fit_their_bits(plan, bn, nqb):
    top = 1 << plan.row_bits()
    sizes = [1024, 16384, 100_003, 1_000_000] + [
        m * top + e for m in (1, 2, 3, 17, 63) for e in (-4 * bn, -bn, -1, 0, 1, bn, 5 * bn)]
    for nb in sizes + [2**31 - 1 - e for e in (0, 1, bn - 1, bn, 2 * bn)]:
        out = (ctypes.c_int64 * 2)()
        plan.chunks(nqb, nb, bn, out)
        n, length = out
        assert length < top and length % bn == 0, (nqb, nb, length)
        assert (n - 1) * length < nb <= n * length, (nqb, nb, n, length)


# pools and sample scores of a batch of queries: at most 1 GiB each
@pytest.mark.parametrize("keff", [17, 48, 116, 528, 1040])
def test_batches_fit_their_memory(plan, keff):
    for nb in [16384, 100_003, 1 << 20, 10_000_019, 1 << 27, 2**31 - 1]:
        for nq in (1, 64, 1000, 100_000, 10_000_000):
            out = (ctypes.c_int64 * 3)()
            plan.batch(nq, nb, keff, out)
            b, cap, sample = out
            assert min(nq, 64) <= b <= nq
            assert b * cap * 8 <= 1 << 30 and b * sample <= 1 << 30, (nq, nb, keff, b, cap)

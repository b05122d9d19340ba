"""The library's dispatch rules (csrc/pa_route.h, plain C++) compiled for the
host, so that a test can state which kernel a call takes."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_09345_amd", "csrc")

_SOURCE = """
#include "pa_route.h"
extern "C" int blocks(int s, int H_kv, int rows, int seqs, int cus) { return pa::prefill_blocks(s, H_kv, rows, seqs, cus); }
extern "C" int to_split(int s, int H_kv, int rows, int seqs, int max_q, int max_ctx, int cus) {
  return pa::chunks64_to_split({s, H_kv, rows, seqs, max_q, max_ctx}, cus);
}
"""


@functools.cache
def _lib():
    d = tempfile.mkdtemp()
    src, so = os.path.join(d, "route.cpp"), os.path.join(d, "route.so")
    with open(src, "w") as f:
        f.write(_SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
    return ctypes.CDLL(so)


def prefill_blocks(s, H_kv, rows, seqs, cus=256):
    return _lib().blocks(s, H_kv, rows, seqs, cus)


def chunks64_to_split(s, H_kv, rows, seqs, max_q, max_ctx, cus=256):
    return bool(_lib().to_split(s, H_kv, rows, seqs, max_q, max_ctx, cus))


def takes_split(b, cus=256):
    """Whether a bf16 head_dim 64 varlen batch's chunks take the split-K kernel."""
    s, H_kv = b.q.shape[1] // b.k_pages.shape[1], b.k_pages.shape[1]
    return chunks64_to_split(s, H_kv, b.num_q_rows, b.num_seqs, int(b.q_lens.max()), int(b.context_lens.max()), cus)


def takes_blocks(b, cus=256):
    """16-row blocks per wave of the prefill kernel for a varlen batch."""
    s, H_kv = b.q.shape[1] // b.k_pages.shape[1], b.k_pages.shape[1]
    return prefill_blocks(s, H_kv, b.num_q_rows, b.num_seqs, cus)

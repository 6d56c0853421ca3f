"""What the attention entry points hand to their kernels, without a GPU: in a process of its own the library's launches go to a
recorder that stands in for the HIP runtime's launch call and notes the pointers a kernel would be given."""
import ctypes
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# The second argument of every attention kernel is AttnArgs (csrc/kernels.h), whose sixth pointer is k_idx.
RECORDER = r"""
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim3_t;
static dim3_t g, b;
static size_t lds;
static void* st;
int n_launches = 0;
void* k_idx[8];
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t bytes, void* stream) { g = grid; b = block; lds = bytes; st = stream; return 0; }
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* bytes, void** stream) { *grid = g; *block = b; *bytes = lds; *stream = st; return 0; }
int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t bytes, void* stream) {
  if (n_launches < 8) k_idx[n_launches++] = ((void**)args[1])[5];
  return 0;
}
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipFuncSetAttribute(const void* f, int attr, int value) { return 0; }
int hipGetLastError(void) { return 0; }
"""


def _recorded(recorder, dtype, d, batch, chunk, max_budget, sparse, list_at, count_at):
    """The k_idx of each launch of one call whose other pointers are placeholders that nothing follows."""
    import paper_2602_08722_amd as pk
    from tests.test_abi import _shape
    lib = pk.load_library()
    s = _shape(pk, dtype=dtype, head_dim=d, batch=batch, chunk_len=chunk, max_budget=max_budget)
    at, ws, big = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x10000), ctypes.c_size_t(1 << 40)
    ctypes.c_int.in_dll(recorder, "n_launches").value = 0
    if sparse:
        st = lib.quoka_sparse_attn(ctypes.byref(s), at, at, at, ctypes.c_void_p(list_at), ctypes.c_void_p(count_at), at, at, at, None, ws, big, None)
    else:
        st = lib.quoka_dense_attn(ctypes.byref(s), at, at, at, ctypes.c_void_p(count_at), at, at, at, None, ws, big, None)
    assert st == 0
    n = ctypes.c_int.in_dll(recorder, "n_launches").value
    return list((ctypes.c_void_p * 8).in_dll(recorder, "k_idx"))[:n]


# float32: units, and a wave a row; bfloat16: decode of one sequence and of a batch, blocks of row blocks
FORMS = [(0, 64, 1, 64), (0, 128, 2, 33), (0, 128, 1, 2), (1, 128, 1, 1), (1, 64, 2, 8), (1, 128, 1, 9), (1, 64, 1, 300), (1, 128, 1, 8192)]


def check_lists(recorder_path):
    recorder = ctypes.CDLL(recorder_path, mode=ctypes.RTLD_GLOBAL)   # ahead of everything that brings the HIP runtime
    lists, counts = 0x2004, 0x3000
    for form in FORMS:
        got = _recorded(recorder, *form, 0, True, lists, counts)
        assert got and set(got) == {counts}, (form, got)
        got = _recorded(recorder, *form, 0, True, None, counts)
        assert got and set(got) == {counts}, (form, got)
        got = _recorded(recorder, *form, 100, True, lists, counts)
        assert got and set(got) == {lists}, (form, got)
        got = _recorded(recorder, *form, 100, False, None, counts)
        assert got and set(got) == {None}, (form, got)


def test_an_empty_key_list_is_never_handed_to_a_kernel(tmp_path):
    """k_idx [b, n_KV, 0] has no entry, and the kernels fetch a list's entries before they know its length: with max_budget == 0 they
    are given k_cnt in its place, whatever k_idx is; a list with room for entries as it is, and none for dense calls."""
    (tmp_path / "recorder.c").write_text(RECORDER)
    so = str(tmp_path / "recorder.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", so, str(tmp_path / "recorder.c")], check=True)
    r = subprocess.run([sys.executable, "-c", f"import sys; sys.path.insert(0, {ROOT!r}); from tests.test_launch_arguments import check_lists; "
                                              f"check_lists({so!r})"], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]

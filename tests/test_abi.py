"""The C ABI on a host without a GPU: the library loads, exports every entry
point include/kkm.h declares, and rejects bad arguments before any device work."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "kkm.h")


def declared():
    txt = open(HEADER).read()
    return sorted(set(re.findall(r"^(?:kkm_status|size_t|int64_t|const char \*)\s*(kkm_\w+)\(", txt, re.M)))


@pytest.fixture(scope="module")
def lib():
    import paper_2501_05587_amd as kkm
    return kkm.lib()


def test_every_declared_symbol_is_exported(lib):
    names = declared()
    assert {"kkm_gram", "kkm_iterate", "kkm_fit"} <= set(names)
    for nm in names:
        assert hasattr(lib, nm), nm


def test_binding_names_match_header():
    import paper_2501_05587_amd as kkm
    assert set(kkm.EXPORTS) == set(declared())


def test_argument_validation_without_device_work(lib):
    vp = ctypes.c_void_p
    # kkm_gram: n = 0
    assert lib.kkm_gram(None, 0, 4, 4, 2, 1.0, 0.0, 1, 0, 0, None, 0, None, None, 0, None) == -1
    assert b"bad sizes" in lib.kkm_last_error()
    # Gaussian with gamma <= 0 and a bad degree
    fake = vp(16)
    assert lib.kkm_gram(fake, 8, 4, 4, 2, -1.0, 0.0, 1, 0, 0, fake, 8, fake, None, 0, None) == -1
    assert lib.kkm_gram(fake, 8, 4, 4, 1, 1.0, 1.0, 0, 0, 0, fake, 8, fake, None, 0, None) == -1
    assert lib.kkm_gram(fake, 8, 4, 4, 7, 1.0, 1.0, 1, 0, 0, fake, 8, fake, None, 0, None) == -1
    # ldx < d, ldk < n
    assert lib.kkm_gram(fake, 8, 4, 3, 2, 1.0, 0.0, 1, 0, 0, fake, 8, fake, None, 0, None) == -1
    assert lib.kkm_gram(fake, 8, 4, 4, 2, 1.0, 0.0, 1, 0, 0, fake, 7, fake, None, 0, None) == -1
    # a BF16 product whose 128 rounded rows pass a 32-bit buffer range
    big_d = 9_000_000
    assert lib.kkm_gram(fake, 8, big_d, big_d, 2, 1.0, 0.0, 1, 1, 0, fake, 8, fake, fake,
                        ctypes.c_size_t(1 << 40), None) == -5
    assert b"too large" in lib.kkm_last_error()
    # kkm_iterate: k > n, aliasing, k too large
    z = None
    assert lib.kkm_iterate(fake, 0, 8, fake, 8, 9, fake, 0, vp(32), fake, fake, fake, z, z, z, 0, z) == -1
    assert lib.kkm_iterate(fake, 0, 8, fake, 8, 2, fake, 0, fake, fake, fake, fake, z, z, z, 0, z) == -1
    assert lib.kkm_iterate(fake, 0, 5000, fake, 5000, 2000, fake, 0, vp(32), fake, fake, fake, z, z,
                           z, 0, z) == -5
    assert lib.kkm_iterate(fake, 0, 8, fake, 8, 2, fake, 9, vp(32), fake, fake, fake, z, z, z, 0, z) == -1
    # kkm_fit: k = 0, negative max_iter
    J = ctypes.c_double()
    it = ctypes.c_int32()
    assert lib.kkm_fit(fake, 8, 4, 4, 0, 2, 1.0, 0.0, 1, fake, 5, 1, fake, ctypes.byref(J),
                       ctypes.byref(it), None, 0, None) == -1
    assert lib.kkm_fit(fake, 8, 4, 4, 2, 2, 1.0, 0.0, 1, fake, -1, 1, fake, ctypes.byref(J),
                       ctypes.byref(it), None, 0, None) == -1


def test_workspace_sizes(lib):
    import paper_2501_05587_amd as kkm
    assert kkm.iterate_workspace_bytes(0, 3) == 0
    small = kkm.iterate_workspace_bytes(1000, 4)
    big = kkm.iterate_workspace_bytes(200000, 64)
    assert 0 < small < big
    # partial sums stay a small fraction of the n x n matrix they summarise
    assert big < 0.002 * 200000 ** 2 * 4
    assert kkm.gram_workspace_bytes(1000, 16) >= 1000 * 4


def test_matfree_workspace_size_of_the_longest_rows_serves_shorter_ones():
    # the FP32 product reads the caller's rows: what a step needs depends on n and
    # k alone, whichever sweep the row length takes
    import paper_2501_05587_amd as kkm
    for n, k in ((1, 1), (100, 3), (4097, 16), (50000, 32), (200000, 64)):
        sizes = [kkm.matfree_workspace_bytes(n, d, k, kkm.F32) for d in (1, 32, 33, 256, 257, 1000)]
        assert len(set(sizes)) == 1, (n, k, sizes)
    # a buffer of the size that the sweep of longer rows has always asked for
    assert kkm.matfree_workspace_bytes(50000, 128, 32, kkm.F32) <= 12374784


def test_instance_struct_layout_matches_header(tmp_path):
    """The ctypes mirror of kkm_instance has the C struct's size and offsets."""
    import subprocess

    import paper_2501_05587_amd as kkm
    src = tmp_path / "layout.c"
    fields = [f[0] for f in kkm.KkmInstance._fields_]
    src.write_text('#include <stdio.h>\n#include <stddef.h>\n#include "kkm.h"\nint main(void) {\n'
                   '  printf("%zu\\n", sizeof(kkm_instance));\n' +
                   "".join('  printf("%%zu\\n", offsetof(kkm_instance, %s));\n' % f for f in fields) +
                   "  return 0;\n}\n")
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c99", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)],
                   check=True)
    got = [int(x) for x in subprocess.run([str(exe)], check=True, capture_output=True,
                                          text=True).stdout.split()]
    want = [ctypes.sizeof(kkm.KkmInstance)] + [getattr(kkm.KkmInstance, f).offset for f in fields]
    assert got == want


def test_batched_validation_without_device_work(lib):
    import paper_2501_05587_amd as kkm
    I = kkm.KkmInstance
    fake = 4096

    def arr(*ps):
        a = (I * len(ps))()
        for i, p in enumerate(ps):
            a[i] = p
        return a

    ok = I(fake, 100, 8, 8, 5, 2, 0.5, 0.0, 1, 0)
    bad_k = I(fake, 10, 8, 8, 11, 2, 0.5, 0.0, 1, 0)
    big_k = I(fake, 5000, 8, 8, 2000, 2, 0.5, 0.0, 1, 0)
    bad_chunk = I(fake, 100, 8, 8, 5, 2, 0.5, 0.0, 1, -3)
    bad_gamma = I(fake, 100, 8, 8, 5, 2, -1.0, 0.0, 1, 0)
    obj = (ctypes.c_double * 2)()
    its = (ctypes.c_int32 * 2)()
    vp = ctypes.c_void_p

    def fit(a, count, **kw):
        return lib.kkm_fit_batched(a, count, kw.get("gp", 0), kw.get("ks", 0), kw.get("ep", 0),
                                   vp(fake), kw.get("mi", 5), 1, 1, vp(fake), obj, its, None,
                                   None, 0, None)

    assert fit(arr(ok), 0) == -1
    assert fit(arr(ok, bad_k), 2) == -1
    assert b"problem 1" in lib.kkm_last_error()
    assert fit(arr(big_k), 1) == -5
    assert fit(arr(bad_chunk), 1) == -1
    assert fit(arr(ok, bad_gamma), 2) == -1
    assert b"problem 1" in lib.kkm_last_error() and b"gamma" in lib.kkm_last_error()
    assert fit(arr(ok), 1, gp=5) == -1
    assert fit(arr(ok), 1, ep=7) == -1
    assert fit(arr(ok), 1, mi=-1) == -1
    # workspace sizing is host arithmetic: every K is kept, rows padded to 64
    ws = lib.kkm_fit_batched_workspace_bytes
    one = ws(arr(ok), 1, 0, 0)
    assert one >= 100 * 128 * 4
    assert ws(arr(ok, ok), 2, 0, 0) >= 2 * 100 * 128 * 4
    assert ws(arr(ok), 1, 1, 1) < one          # BF16 K is half the size
    assert ws(arr(bad_k), 1, 0, 0) == 0


def test_training_step_numbers_past_the_largest_are_refused(lib):
    # Adam's step numbers are t0 + 1 .. t0 + steps: the first is already past int32
    vp, cs = ctypes.c_void_p, ctypes.c_size_t
    fake = vp(4096)
    for B in (8, 256):
        need = lib.kkm_mlp_train_fresh_workspace_bytes(B, 4, 5, 6, 3)
        assert lib.kkm_mlp_train_fresh(fake, fake, fake, 4, 5, 6, 3, fake, 4, B, 1, 2147483647, 2, 1.0, 0.0, 1, 1e-3,
                                       0.9, 0.999, 1e-8, fake, fake, cs(need), None) == -1
        assert b"bad arguments" in lib.kkm_last_error()

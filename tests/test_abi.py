"""CPU-side checks of the boundary: the library loads and exports every symbol the header declares."""
import os
import re

import paper_2310_03841_amd as ab

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "abft.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(abft_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = _declared()
    assert "abft_gemm" in names and "abft_verify" in names and "abft_correct" in names and "abft_inject" in names
    L = ab.lib()
    for n in names:
        assert hasattr(L, n), n
    assert names == ab.exported_symbols()


def test_strerror_and_version_and_tile_shape():
    assert ab.abft_version() >= 100
    for code in (0, -1, -2, -3, -4, -5, -6):
        assert ab.abft_strerror(code) not in ("", "unknown error")
    tm, tn = ab.abft_tile_shape(ab.ABFT_BF16, ab.make_shape(12608, 3072, 768))
    assert tm % 32 == 0 and tn % 32 == 0


def test_struct_layout_matches_header():
    import ctypes
    assert ctypes.sizeof(ab.abft_shape) == 11 * 8
    assert ctypes.sizeof(ab.abft_config) == 5 * 8
    assert ctypes.sizeof(ab.abft_result) == 4 * 8


def test_items_side_by_side_in_wide_rows_take_the_item_kernel():
    """An item is one workgroup's (its tile is the whole of it) as long as its rows, times the bytes between them, fit 32-bit offsets: q, k and v of
    16 heads x 64 for 86 images and more, as rows of one tensor.  The line falls with the rows that are read."""
    def whole(dtype, M, N, K, trans_b, items, pitch_bytes):
        es = 1 if dtype == ab.ABFT_I8 else 2
        ld = pitch_bytes // es
        s = ab.make_shape(M, N, K, batch=items, lda=K + 64, ldb=ld, ldc=640, strideA=M * (K + 64), strideB=64, strideC=M * 640, transB=trans_b)
        return ab.abft_tile_shape(dtype, s) == (M, N)

    for images in (85, 86, 128, 256, 320):
        pitch = images * 16 * 3 * 64 * 2
        assert whole(ab.ABFT_BF16, 577, 577, 64, True, 16 * images, pitch), images
        assert whole(ab.ABFT_BF16, 197, 64, 200, False, 16 * images, pitch), images
    for M, N, K, trans_b in ((577, 577, 64, True), (197, 197, 64, True), (197, 64, 200, False), (64, 128, 320, True)):
        rows = N if trans_b else K
        assert whole(ab.ABFT_I8, M, N, K, trans_b, 64, 1 << 20)
        assert not whole(ab.ABFT_I8, M, N, K, trans_b, 64, ((1 << 31) // rows + 15) // 16 * 16)

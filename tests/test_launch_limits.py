"""Limits that launchers check before any launch (no GPU needed)."""
import ctypes as C
import subprocess

import paper_2510_02345_amd as cm

HIP_ERROR_INVALID_VALUE = 1


def _internal(name):
    names = subprocess.run(["nm", "-D", "--defined-only", cm.binding.lib_path()], check=True, capture_output=True,
                           text=True).stdout.split()
    return getattr(cm.lib(), next(n for n in names if name in n))


def test_quantiser_takes_a_thread_per_word_only_while_a_launch_has_as_many():
    f = _internal("quantize_by_words")
    f.restype, f.argtypes = C.c_bool, [C.c_long, C.c_int, C.c_int]
    for q in (8, 64, 512):
        assert f(1, 512, q) and f((1 << 26) - 4, 512, q)
        assert not f(1 << 26, 512, q) and not f(1 << 33, 512, q)     # 2^32 words and more
    assert not f(1, 96, 24) and not f(1, 1024, 1024) and not f(1, 64, 2)


def test_grouped_product_takes_no_more_groups_than_lanes():
    f = _internal("launch_gemm_plain")
    P, I, L = C.c_void_p, C.c_int, C.c_long
    f.restype = I
    # W, w_gstride, ldw, N, X, ldx, gather, x_div, Kc, offsets, n_groups, rows, krange, rowmap, out, ldo, out_f32, stream,
    # kstep_w, kstep_x
    f.argtypes = [P, L, I, I, P, I, P, I, I, P, I, I, P, P, P, I, C.c_bool, P, L, L]
    for N in (32, 256):   # the thin and the tiled product
        for out_f32 in (False, True):
            assert f(None, 0, 64, N, None, 64, None, 1, 64, None, 65, 0, None, None, None, N, out_f32, None, 0, 0) == HIP_ERROR_INVALID_VALUE


class _Dims(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("d", "d_ff", "G", "K", "r", "k", "q", "KR", "KRp")]


def test_weight_streams_take_passes_of_64_tokens_where_they_save_a_reading_and_fill_the_chip():
    f = _internal("stream_cols")
    f.restype, f.argtypes = C.c_int, [C.POINTER(_Dims), C.c_int, C.c_bool]

    def cols(d, d_ff, G, T, down):
        return f(_Dims(d, d_ff, G, 8, 16, 2, 64, 128, 128), T, down)

    for T in range(17, 33):                       # one cluster: 32 tokens are one pass in either form
        assert cols(4096, 14336, 1, T, False) == 32 and cols(4096, 14336, 1, T, True) == 32
    assert cols(4096, 14336, 1, 65, False) == 64 and cols(4096, 14336, 1, 65, True) == 64
    assert cols(4096, 14336, 1, 64, True) == 32   # 32 row blocks in four parts: 128 workgroups
    assert cols(8192, 8192, 1, 64, False) == 32   # 64 workgroups
    assert cols(4096, 14336, 3, 60, False) == 32 and cols(2048, 8192, 5, 100, False) == 32   # 336 and 320 for 256 CUs
    assert cols(4096, 14336, 3, 96, False) == 64
    for G in (2, 4, 8):
        for T in range(18 * G + 1, 257):
            assert cols(4096, 14336, G, T, False) == 64
            assert cols(4096, 14336, G, T, True) == (64 if T > 28 * G else 32)
    assert cols(1024, 4096, 4, 256, False) == 32  # a base that the caches keep


def test_permutation_that_cannot_take_t1_along_is_refused():
    f = _internal("launch_sort_pairs_t1")
    P, I = C.c_void_p, C.c_int
    # dims, cluster_id, expert_idx, T, x, x_div, v1cat, t1, perm, inv_perm, offsets, counts, rowmap, perm2, stream
    f.restype, f.argtypes = I, [C.POINTER(_Dims), P, P, I, P, I, P, P, P, P, P, P, P, P, P]
    dims = _Dims(64, 64, 64, 100, 4, 2, 64, 400, 416)   # 6400 bins, more than a layer has and than fit its LDS
    assert f(dims, None, None, 300, None, 1, *[None] * 9) == HIP_ERROR_INVALID_VALUE


class _Compress(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("out_dim", "in_dim", "G", "K", "r", "q_group", "sketch", "n_iter", "use_gate")] + [("gate_gamma", C.c_float)]


def test_error_pass_takes_four_row_tiles_a_workgroup_where_the_last_has_enough_of_them():
    f = _internal("error_row_tiles")
    f.restype, f.argtypes = C.c_int, [C.POINTER(_Compress)]

    def tiles(out_dim, in_dim, experts, r):
        return f(_Compress(out_dim, in_dim, experts // 8, 8, r, 32, r + 8, 2, 0, 0.0))

    assert tiles(8192, 2048, 64, 16) == 4 and tiles(8192 + 64, 2048, 64, 16) == 4
    assert tiles(512, 2048, 64, 16) == 4 and tiles(448, 2048, 128, 16) == 4
    for out_dim in (320, 384, 576, 832, 1088):
        assert tiles(out_dim, 2048, 128, 16) == 1, out_dim
    assert tiles(384, 2048, 128, 32) == 4 and tiles(1088, 2048, 64, 32) == 4 and tiles(320, 2048, 128, 32) == 1
    assert tiles(4096, 1024, 8, 16) == 1     # two workgroups a CU
    assert tiles(8192, 128, 64, 16) == 1     # narrower than four column tiles

"""Which tiles the library's launchers take, asked on the host (the functions are the library's own, not of its C ABI; the
operand addresses are never read)."""
import ctypes as C

import paper_2503_02550_amd as S

# rows, columns, blocks of a CU at a time; the library's order
TILES = {"32x64": (32, 64, 3), "64x64": (64, 64, 2), "128x64": (128, 64, 2), "128x128 one": (128, 128, 1), "128x128 two": (128, 128, 2),
         "256x128": (256, 128, 1), "256x256": (256, 256, 1)}


def takes(a, name):
    """Whether the rows that the library counts for a round of the product's tiles are those of the named tiles and of no
    others."""
    rows = getattr(S.lib, "_ZN3sif15gemm_round_rowsERK13sif_gemm_args")
    rows.restype, rows.argtypes = C.c_uint32, [C.POINTER(S.sif_gemm_args)]
    got = rows(a)
    return [t for t, (bm, bn, slots) in TILES.items() if got == bm * max(1, 256 * slots // ((a.n + bn - 1) // bn))] == [name]


def group(products):
    """(tiles with their padding, name of the tiles) of a launch over several products."""
    fill = getattr(S.lib, "_ZN3sif15gemm_group_fillEPK13sif_gemm_argsjPvPNS_9GemmGroupE")
    fill.restype, fill.argtypes = C.c_int, [C.c_void_p, C.c_uint32, C.c_void_p, C.c_void_p]
    n, got = len(products), (C.c_uint32 * 3)()
    assert fill((S.sif_gemm_args * n)(*products), n, (C.c_char * S.sif_k_gemm_bf16_group_bytes(n))(), got) == 0
    return got[0], list(TILES)[got[1]]


def part(products, first):
    """How many of the products one launch holds where those from `first` on could follow it."""
    f = getattr(S.lib, "_ZN3sif15gemm_group_partEPK13sif_gemm_argsjj")
    f.restype, f.argtypes = C.c_uint32, [C.c_void_p, C.c_uint32, C.c_uint32]
    return f((S.sif_gemm_args * len(products))(*products), first, len(products))

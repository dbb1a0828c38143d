"""Which tiles the library's launchers take, asked on the host (the functions are the library's own, not of its C ABI; the
operand addresses are never read)."""
import ctypes as C

import paper_2503_02550_amd as S

# the library's order
TILES = ["32x64", "64x64", "128x64", "128x128 one", "128x128 two", "256x128", "256x256"]
KERNELS = TILES + ["fetching 32x64", "fetching 64x64", "fetching 128x64", "fetching 32x32"]


def kernel(a):
    """The kernel that the launcher takes for a product: the ring or ping-pong kernel of its tiles, or the one with wavefronts
    that only fetch."""
    f = getattr(S.lib, "_ZN3sif14gemm_kernel_ofERK13sif_gemm_args")
    f.restype, f.argtypes = C.c_int, [C.POINTER(S.sif_gemm_args)]
    return KERNELS[f(a)]


def group(products):
    """(tiles with their padding, name of the tiles) of a launch over several products."""
    fill = getattr(S.lib, "_ZN3sif15gemm_group_fillEPK13sif_gemm_argsjPvPNS_9GemmGroupE")
    fill.restype, fill.argtypes = C.c_int, [C.c_void_p, C.c_uint32, C.c_void_p, C.c_void_p]
    n, got = len(products), (C.c_uint32 * 3)()
    assert fill((S.sif_gemm_args * n)(*products), n, (C.c_char * S.sif_k_gemm_bf16_group_bytes(n))(), got) == 0
    return got[0], TILES[got[1]]


def part(products, first):
    """How many of the products one launch holds where those from `first` on could follow it."""
    f = getattr(S.lib, "_ZN3sif15gemm_group_partEPK13sif_gemm_argsjj")
    f.restype, f.argtypes = C.c_uint32, [C.c_void_p, C.c_uint32, C.c_uint32]
    return f((S.sif_gemm_args * len(products))(*products), first, len(products))

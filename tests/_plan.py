"""The library's GEMM tile plan (plan_gemm, an internal host function) for tests
that name the kernel instance they mean to run."""

import ctypes as C

from paper_2609_36722_amd import _lib

BF16, F32 = 0, 3             # epilogue modes
SPLIT, FEW, DOWN = 1, 2, 4   # what a caller allows: key splits, the 32-token tiles, t by a kernel of its own

# the launcher's tiles (tokens x features); a: read-ahead, k: two k-groups
TILES = ["256x256a", "256x192a", "128x256a", "128x128a", "128x64a", "128x128", "64x96", "64x64", "128x192k", "128x96k",
         "32x128a", "32x64a", "128x256"]
FUSES = {"128x256", "128x128", "64x96", "64x64", "128x192k", "128x96k"}   # compute a low-rank t of up to 32 ranks
KERNELS = {"a": "gemm_ahead_kernel", "k": "gemm_kg2_kernel"}


class _Plan(C.Structure):
    _fields_ = [("tile", C.c_int), ("n_split", C.c_int), ("kt_split", C.c_int)]


def plan_gemm(n_tok, n_out, k_dim, r_pad, may, mode=BF16):
    fn = getattr(_lib.lib(), "_ZN7attuner9plan_gemmEiiiiii")
    fn.restype, fn.argtypes = _Plan, [C.c_int] * 6
    p = fn(n_tok, n_out, k_dim, r_pad, mode, may)
    return p.tile, p.n_split, p.kt_split


def plain_plan(n_tok, n_out, k_dim, mode=BF16):
    """"tile/splits" of a plain product, "gemv" for the GEMV."""
    tile, n_split, _ = plan_gemm(n_tok, n_out, k_dim, 0, SPLIT | FEW, mode)
    return f"{TILES[tile]}/{n_split}" if tile >= 0 else "gemv"


def qproj_plan(n_tok, n_out, k_dim, rank):
    """The tile of an adapted projection, "gemv" for the GEMV."""
    tile, _, _ = plan_gemm(n_tok, n_out, k_dim, (rank + 15) // 16 * 16, DOWN)
    return TILES[tile] if tile >= 0 else "gemv"


def kernel_of(plan):
    """The kernel that runs a plan other than the GEMV."""
    return KERNELS.get(plan.split("/")[0][-1], "gemm_lora_kernel")

"""Sizes that reach each GEMM kernel of the scaled matmul on 256 CUs, so that
the GPU tests name the kernel that they mean to run. The names are those of
host_gemm_choice.cpp: wave (16 to 64 x 64 tiles), pair (128 x 128, two
workgroups to a CU), mid128 and mid256 (128 x 128 and 128 x 256, one to a CU),
big (256 x 256, 4 waves; with block scales of A [K][M] and B [K][N], 8 waves),
fused8 (256 x 256, 8 waves, fused epilogue); "-rounds" where a workgroup takes
more than one tile. test_gemm_choice_host.py checks every entry against the
library's rule."""
from __future__ import annotations

# plain calls: ragged in M, N and K, and with every tile inside the matrix
PLAIN = {"pair": (700, 1500, 255), "mid128": (700, 1500, 4100), "mid256": (1100, 4000, 4100),
         "big": (2100, 4100, 200), "big-rounds": (4200, 4200, 200)}
PLAIN_INSIDE = {"wave": (512, 384, 256), "big": (2304, 4096, 256)}
# with a residual, an activation or channel scales
FUSED = {"pair": (700, 1500, 255), "mid128": (700, 1500, 4100), "mid256": (1100, 4000, 4100),
         "pair-rounds": (4100, 4200, 400), "fused8": (2100, 4100, 200)}
# with block scales
MX = {"wave-rounds": (800, 2100, 200), "big": (1100, 2100, 200), "big-rounds": (4200, 4200, 200)}
MX_INSIDE = {"wave-rounds": (384, 4096, 256), "big": (1280, 2304, 512)}
# plain calls: big with a statistic, pair without one
SHORT_K = [(2048, 4096, 400), (2000, 4000, 250)]

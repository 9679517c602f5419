"""Which step a system takes (the options "fused_active" and "brick_active"),
decided on the host: lattices that fill the brick step's bricks take it, those
that leave them partly empty (thin films, rods, cut bricks) or have too many
keep the two-launch step."""
import numpy as np
import pytest

import paper_1310_6143_amd as sl

P, FILM = (1, 1, 1), (1, 1, 0)


def _routes(kind, dims, periodic, prec, fused=1):
    csr = sl.build_sc(dims, periodic) if kind == "sc" else sl.build_bcc(dims, periodic, kind == "bcc14")
    with sl.SpinSystem(len(csr[0]) - 1, precision=prec) as s:
        s.set_option("check_symmetry", 0)
        s.set_option("fused", fused)
        s.set_neighbours(csr[0], csr[1], csr[2], [6e-21, 3e-21] if kind == "bcc14" else [6e-21])
        s.set_lattice(1 if kind == "sc" else 2, dims, periodic)
        s.set_materials(1e-23, 0.0, [0.0, 0.0, 1.0])
        return s.get_option("brick_active"), s.get_option("fused_active")


# (kind, cells, periodic, brick step in FP32, in FP64)
CASES = [("sc", (5, 5, 5), P, 1, 1), ("sc", (64, 64, 64), P, 1, 1), ("sc", (64, 64, 1), FILM, 1, 1),
         ("sc", (256, 256, 1), FILM, 1, 1), ("sc", (512, 512, 1), FILM, 0, 0), ("sc", (512, 512, 2), FILM, 0, 0),
         ("sc", (5, 5, 4000), P, 1, 0), ("sc", (5, 5, 20000), P, 0, 0), ("sc", (9, 9, 6000), P, 0, 0),
         ("bcc8", (33, 33, 33), P, 1, 1), ("bcc8", (64, 64, 64), P, 1, 1), ("bcc8", (128, 128, 1), FILM, 1, 1),
         ("bcc8", (512, 512, 1), FILM, 0, 0), ("bcc8", (9, 5, 8000), P, 0, 0),
         ("bcc14", (32, 32, 32), P, 1, 1), ("bcc14", (34, 34, 36), P, 0, 0), ("bcc14", (5, 5, 1900), P, 0, 0),
         ("bcc14", (200, 240, 1), FILM, 0, 0)]


@pytest.mark.parametrize("kind,dims,periodic,fp32,fp64", CASES)
def test_bricks_only_where_lattices_fill_them(kind, dims, periodic, fp32, fp64):
    assert _routes(kind, dims, periodic, sl.FP32) == (fp32, 0)
    assert _routes(kind, dims, periodic, sl.FP64) == (fp64, 0)


def test_option_fused_overrides():
    for prec in (sl.FP32, sl.FP64):
        assert _routes("sc", (16, 16, 16), P, prec, 0) == (0, 0)
        assert _routes("sc", (16, 16, 16), P, prec, 2) == (0, 1)

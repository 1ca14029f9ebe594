"""The file of the timed selection (NGF_TUNE_CACHE): lines of the kernels that are
there are used, for the kind of spacing they were timed with; lines of earlier
kernels, and what is no line, are passed over."""

import pytest

pytestmark = pytest.mark.gpu

M = (32, 32, 32)


def _variant(ngf, h):
    import torch
    R = torch.randn(M, device="cuda")
    with ngf.Context(alpha=0.1, tau=1.0, rho=1.0, levels=1) as ctx:
        ctx.build_pyramid(R, R, (h, h, h))
        return ctx.get_kernel(0)


def test_lines_of_the_cache_file(gpu_lib, tmp_path, monkeypatch):
    ngf = gpu_lib
    path = tmp_path / "tune"
    monkeypatch.setenv("NGF_TUNE_CACHE", str(path))
    # 0, the 8 x 8 x 32 tile, takes twice the time of the small one here (8)
    path.write_text("gfx950 32 32 32 n17,17,17 0\nk1 gfx950 32 32 32 n17,17,17 p1 0\nother\n")
    assert _variant(ngf, 1.0) == 8
    lines = path.read_text().splitlines()
    assert len(lines) == 4 and lines[3].startswith("k2 gfx950 32 32 32 n17,17,17 p1 ")
    path.write_text("other\n" + lines[3].rsplit(" ", 1)[0] + " 0\n")
    assert _variant(ngf, 1.0) == 0 and _variant(ngf, 2.0) == 0
    assert _variant(ngf, 0.9) == 8
    assert path.read_text().splitlines()[2].startswith("k2 gfx950 32 32 32 n17,17,17 p0 ")
    path.write_text(path.read_text() + lines[3].rsplit(" ", 1)[0] + " 99\n")
    assert _variant(ngf, 1.0) == 0


def test_a_line_that_does_not_suit_the_grid(gpu_lib, tmp_path, monkeypatch):
    """Only the general pass runs on a node grid without a ratio of 2 or 4."""
    import torch
    ngf = gpu_lib
    path = tmp_path / "tune"
    monkeypatch.setenv("NGF_TUNE_CACHE", str(path))
    path.write_text("k2 gfx950 32 32 32 n11,12,13 p1 8\n")
    R = torch.randn(M, device="cuda")
    with ngf.Context(alpha=0.1, tau=1.0, rho=1.0, levels=1) as ctx:
        ctx.set_node_grid((11, 12, 13))
        ctx.build_pyramid(R, R)
        assert ctx.get_kernel(0) == 14

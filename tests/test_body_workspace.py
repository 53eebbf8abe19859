"""The draft body's workspace: what is enough for a number of rows is enough for fewer."""
import pytest

from paper_2601_20357_amd import binding

# both kinds of head that the one-launch step takes, and others; caches of one and of several key ranges; widths around each limit
SIZES = [(layers, d, hd, d_ff, max_ctx) for layers in (1, 12) for d, hd in ((64, 8), (48, 16), (64, 64), (768, 64), (1024, 128), (1024, 64), (1152, 128), (1536, 64),
                                                                           (2048, 64)) for d_ff in (8, 4 * d, 4104) for max_ctx in (100, 8192)]


@pytest.mark.parametrize("layers,d,hd,d_ff,max_ctx", SIZES)
def test_more_rows_never_need_less(layers, d, hd, d_ff, max_ctx):
    cfg = binding.make_body_cfg(layers=layers, d=d, heads=d // hd, d_ff=d_ff, V=100, max_ctx=max_ctx)
    rows = list(range(1, 1100)) + [2000, 5000, 6400, 6401, 20000, 65535]
    need = [binding.tabed_body_workspace_bytes(cfg, r) for r in rows]
    assert need[0] > 0
    assert all(a <= b for a, b in zip(need, need[1:])), next((r, a, b) for r, a, b in zip(rows, need, need[1:]) if a > b)

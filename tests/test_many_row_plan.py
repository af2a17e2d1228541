"""Which kernel shapes the many-row products of test_gpu_parity.MANY_ROWS reach (host arithmetic, no GPU): a change of the
cost model that moves a shape to another plan fails here instead of silently taking a kernel out of that test."""
import ctypes as C

import pytest

from test_gpu_parity import MANY_ROWS, _many_rows_model


def _plan(rows, k, n, swiglu):
    from paper_2605_01106_amd import binding
    tiles, splits = C.c_int(), C.c_int()
    binding.lib.hh_many_row_plan(rows, k, n, int(swiglu), C.byref(tiles), C.byref(splits))
    return tiles.value, splits.value


def _products(cfg):
    d_inproj = 2 * cfg.d_inner + 2 * cfg.d_state + cfg.m_heads + cfg.d_q + 2 * cfg.d_kv
    return {"in": (cfg.d_model, d_inproj), "o": (cfg.d_q, cfg.d_model), "out": (cfg.d_inner, cfg.d_model),
            "up": (cfg.d_model, cfg.d_ff), "down": (cfg.d_ff, cfg.d_model)}


@pytest.mark.parametrize("shape,plans", MANY_ROWS)
def test_plans_are_the_listed_ones(shape, plans):
    sequences, tokens, d_model, d_ff = shape
    got = {name: _plan(sequences * tokens, k, n, name == "up")
           for name, (k, n) in _products(_many_rows_model(d_model, d_ff)).items()}
    assert got == plans


def test_listed_plans_cover_the_kernel():
    epilogue = {"in": "store", "o": "store", "out": "add", "down": "add", "up": "swiglu"}
    nearly_empty, split, handed = set(), set(), set()
    for (sequences, tokens, _, d_ff), plans in MANY_ROWS:
        row_tiles = (sequences * tokens + 15) // 16
        for name, (tiles, splits) in plans.items():
            if 0 < row_tiles % (2 * tiles) <= max(1, tiles // 2):
                nearly_empty.add((epilogue[name], tiles))
            if splits > 1:
                split.add(epilogue[name])
        handed.add(plans["up"][1] == 1 and d_ff % 32 == 0)
    assert nearly_empty == {(e, t) for e in ("store", "add", "swiglu") for t in range(2, 7)}
    assert split == {"store", "add", "swiglu"} and handed == {True, False}

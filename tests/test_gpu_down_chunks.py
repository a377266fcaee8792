"""The down-projection on the matrix cores (3-8 tokens) over every number of
32-row chunks: one 512-column tile, 200 rows per block, and masks that keep a
different number of each block's rows, so that one call has blocks of 0 to 7
chunks with the last one full, one row short and one row long (the last chunks
run code of their own that requests nothing behind them).  Without W_up the same
call has shares of 0 to 200 rows, odd ones among them, for the waves that take
two rows at a time.
"""

import numpy as np
import pytest
import torch

import oracle
import paper_2411_12692_amd as si
from h3check import check_h3, fp16_rows, workspace_ok

pytestmark = pytest.mark.gpu

DEV = "cuda"
KEPT = [0, 1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 160, 161, 192, 193, 200]


@pytest.mark.parametrize("b,gated", [(3, True), (4, True), (8, True), (3, False), (8, False)])
def test_every_number_of_chunks(b, gated):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    R, d = 200, 512
    k = R * cus
    rng = np.random.default_rng(b)
    bits = lambda *s: (rng.standard_normal(s, dtype=np.float32) * 0.05).astype(np.float16).view(np.uint16)  # noqa: E731
    wg, wu, wd, x = bits(k, d), bits(k, d), bits(d, k), bits(b, d)
    dev = lambda a: torch.from_numpy(a.view(np.int16)).to(DEV)  # noqa: E731
    g = si.MLPLayer(dev(wg), dev(wu) if gated else None, dev(wd), max_batch=b)
    assert si._lib.load().si_single_launch(k, d, b) == 1
    mask = np.zeros((cus, R), np.uint8)
    for blk in range(cus):
        mask[blk, rng.permutation(R)[: KEPT[blk % len(KEPT)]]] = 1
    mask = mask.reshape(-1)
    y = g.sparse_mlp(dev(x), mask=torch.from_numpy(mask).to(DEV))
    assert workspace_ok(g.workspace)
    ref = oracle.sparse_mlp(wg, wu, wd, x, mask) if gated else oracle.relu_mlp(wg, wd, x, mask)
    check_h3(g.workspace, k, d, b, mask, ref["h3" if gated else "h"], oracle.fp16_to_f64(x), fp16_rows(wg),
             fp16_rows(wu) if gated else None, ref["g"])
    yr = ref["y"]
    assert np.abs(y.cpu().numpy() - yr).max() <= 1e-4 * np.abs(yr).max()

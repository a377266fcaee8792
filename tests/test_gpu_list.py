"""``si_sparse_mlp`` over a caller's list, as slices of the list per group of
blocks: lists of no row, one row, fewer rows than groups, every row, slices of
more than 512 entries, entries in any order, and entries outside [0, k)
(left out and reported).  y and h3 against the oracle over the same rows, and
the same rows through the mask form, at 1 to 8 tokens.
"""

import numpy as np
import pytest
import torch

import oracle
import paper_2411_12692_amd as si
from h3check import check_h3, fp16_rows, workspace_ok

pytestmark = pytest.mark.gpu

DEV = "cuda"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


class Layer:
    def __init__(self, k, d, b, gated, seed):
        rng = np.random.default_rng(seed)
        bits = lambda *s: (rng.standard_normal(s) * 0.05).astype(np.float16).view(np.uint16)  # noqa: E731
        self.k, self.d, self.b = k, d, b
        self.wg, self.wd, self.x = bits(k, d), bits(d, k), bits(b, d)
        self.wu = bits(k, d) if gated else None
        i16 = lambda a: dev(a.view(np.int16))  # noqa: E731
        self.g = si.MLPLayer(i16(self.wg), i16(self.wu) if gated else None, i16(self.wd), max_batch=b)
        self.xd = i16(self.x)

    def check(self, lst, flags=0, bad=False):
        """The list `lst` (a whole buffer: entries past n are never read as rows)."""
        n = len(lst)
        idx = dev(np.concatenate([lst, np.full(8, 1 << 30)]).astype(np.int32))
        y, cnt = self.g.sparse_mlp(self.xd, active_idx=idx, n_active=dev(np.array([n], np.int32)), flags=flags,
                                   counters=True)
        torch.cuda.synchronize()
        rows = np.array(sorted(r for r in lst if 0 <= r < self.k), dtype=np.int64)
        mask = np.zeros(self.k, np.uint8)
        mask[rows] = 1
        ref = (oracle.sparse_mlp(self.wg, self.wu, self.wd, self.x, mask) if self.wu is not None
               else oracle.relu_mlp(self.wg, self.wd, self.x, mask))
        if rows.size:
            X = oracle.fp16_to_f64(self.x)
            check_h3(self.g.workspace, self.k, self.d, self.b, mask, ref["h3" if self.wu is not None else "h"], X, fp16_rows(self.wg),
                     fp16_rows(self.wu) if self.wu is not None else None, ref["g"])
        if bad:
            assert si.workspace_check(self.g.workspace) == 10  # SI_ERR_LIST, and the workspace is reset
        else:
            assert workspace_ok(self.g.workspace)
        yr, yg = ref["y"], y.cpu().numpy().astype(np.float64)
        assert np.abs(yg - yr).max() <= 1e-4 * max(np.abs(yr).max(), 1e-30)
        n_gate, n_up, n_down = cnt.cpu().numpy().tolist()
        assert n_gate == n and n_up <= n_gate and n_down <= n_gate
        if self.wu is None:
            assert n_up == 0
        ym = self.g.sparse_mlp(self.xd, mask=dev(mask), flags=flags)
        assert np.abs(yg - ym.cpu().numpy()).max() <= 1e-4 * max(np.abs(yr).max(), 1e-30)


@pytest.mark.parametrize("k,d,b,gated", [(1, 128, 1, True), (700, 512, 2, True), (1500, 1152, 3, False),
                                         (900, 2944, 4, True), (1111, 640, 5, True), (2000, 4096, 8, True),
                                         (300, 5120, 1, False), (9000, 8192, 1, True), (1300, 8192, 6, True)])
def test_list_slices(k, d, b, gated):
    L = Layer(k, d, b, gated, 7 * k + d + b)
    rng = np.random.default_rng(k)
    lists = [np.arange(k), np.zeros(0, np.int64), np.array([k - 1]), np.sort(rng.permutation(k)[: max(1, k // 3)]),
             rng.permutation(k)[: max(1, k // 2)]]
    for lst in lists:
        print(f"k={k} d={d} b={b} gated={gated} n={len(lst)}", flush=True)
        L.check(lst)
    L.check(lists[3], flags=si.SI_NO_SPECULATION)
    L.check(lists[3], flags=si.SI_NO_AS)


@pytest.mark.parametrize("b", [1, 4, 7])
def test_list_rows_out_of_range(b):
    k = 1200
    L = Layer(k, 1024, b, True, b)
    lst = np.sort(np.random.default_rng(b).permutation(k)[:400])
    lst[[0, 17, 200, 399]] = [-1, k, 1 << 24, -(1 << 31)]
    L.check(lst, bad=True)
    L.check(lst[1:17])


@pytest.mark.parametrize("b", [1, 3, 8])
def test_list_repeated_rows(b):
    """Each entry of the list counts, also one that repeats a row: next to it
    in an ascending list, or in another group's slice."""
    k = 1200
    L = Layer(k, 1024, b, True, 50 + b)
    rng = np.random.default_rng(b)
    rows = np.sort(rng.permutation(k)[:300])
    twice = rows[::7]
    once, again = np.zeros(k, np.uint8), np.zeros(k, np.uint8)
    once[rows] = 1
    again[twice] = 1
    y1 = oracle.sparse_mlp(L.wg, L.wu, L.wd, L.x, once)["y"]
    yr = y1 + oracle.sparse_mlp(L.wg, L.wu, L.wd, L.x, again)["y"]
    for lst in (np.sort(np.concatenate([rows, twice])), np.concatenate([rows, twice])):
        n = len(lst)
        y, cnt = L.g.sparse_mlp(L.xd, active_idx=dev(lst.astype(np.int32)), n_active=dev(np.array([n], np.int32)),
                                counters=True)
        torch.cuda.synchronize()
        assert workspace_ok(L.g.workspace)
        assert np.abs(y.cpu().numpy() - yr).max() <= 1e-4 * np.abs(yr).max()
        assert cnt.cpu().numpy()[0] == n

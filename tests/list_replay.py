"""The rules by which the list-building threshold kernel keeps a wave's candidate lists, replayed in float64 on the CPU: which
of its branches an input reaches - nothing that the kernel returns would show it, as lists that were pruned, filled or
counted either way give the same thresholds.  The constants are read from the kernel's source, so that an input
whose branch a later constant closes fails the test that needs it."""
import os
import re

import numpy as np

_CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_15180_amd", "csrc")


def constants():
    text = "".join(open(os.path.join(_CSRC, f)).read() for f in ("common.hpp", "fwd_kernels.hpp"))
    names = ("LIST_CAP", "GROW", "GROW_COUNTING", "GROW_HARD", "FIRST_REFRESH", "PRUNE_FROM", "PRUNE_FROM_COUNTING", "MAX_PRUNES", "PRUNE_SUPPORT", "PRUNE_SUPPORT_END",
             "FIRST_TILE_BUSY", "TILE_ENTRIES")
    return {n: int(re.search(r"\b%s = (\d+)" % n, text).group(1)) for n in names}


def _roots(edges, counts, r, h):
    """Roots of f_h (Eq. 9) of rows of counts [R, bins] over the bins' left edges"""
    top = np.where(counts > 0, edges, -np.inf).max(1)
    lo, hi = top - 1.0 - 2 * h, top.copy()
    for _ in range(50):
        mid = 0.5 * (lo + hi)
        up = (counts * np.maximum(edges[None] - mid[:, None], 0.0) ** r).sum(1) >= 1.0
        lo, hi = np.where(up, mid, lo), np.where(up, hi, mid)
    return lo


def replay_wave(X, alpha, nb, **override):
    """X [32, N]: a wave's scores (alpha-1) s, with -inf at keys a causal mask hides.  alpha = 1.5 or 2, where the bound of a refresh is
    the root of the histogram itself."""
    assert X.shape[0] == 32 and X.shape[1] % 64 == 0 and alpha in (1.5, 2.0)
    k = dict(constants(), **override)
    tiles = int(np.isfinite(X).any(0).reshape(-1, 64).any(1).nonzero()[0][-1]) + 1
    r, h = 1.0 / (alpha - 1.0), 1.0 / nb
    bins = np.floor(nb * np.where(np.isfinite(X), X, -1e6)).astype(np.int64)
    first_bin = int(bins.max()) - 4 * nb                     # (nothing listed lies lower in the inputs used here)
    edges = (first_bin + np.arange(4 * nb + 1)) * h
    counts = np.zeros((32, 4 * nb + 1))
    max_count = 0
    lists = [[] for _ in range(64)]                          # (score, bin, counted) by lane; lane = row + 32 half
    run, low, root = np.full(32, -np.inf), np.full(32, -np.inf), np.full(32, -np.inf)
    trig, trig_hard, counting, tight, listed, prunes = k["GROW"], k["GROW_HARD"], False, False, False, 0
    out = dict(counting=False, refreshes=0, prunes=0, pruned=0, prunes_leaving_odd_lists=0, tight_tiles=0, longest=0, overflow=False)
    order = np.arange(64).reshape(8, 8)
    mine = (np.concatenate(order[0::2]), np.concatenate(order[1::2]))      # a lane half's keys of a tile, in register order
    for j in range(tiles):
        x = X[:, 64 * j:64 * j + 64]
        if (x.max(1) >= low).any():
            run = np.maximum(run, x.max(1))
            low = np.maximum(run - 1.0, root)
            if j == 0:
                groups = x.reshape(32, 8, 8).max(2)
                counting = int((groups >= low[:, None]).sum()) >= k["FIRST_TILE_BUSY"]
                if counting:
                    trig_hard = k["GROW_COUNTING"]
            out["tight_tiles"] += tight
            for row in range(32):
                for half in range(2):
                    for key in mine[half]:
                        if x[row, key] >= low[row]:
                            b = int(bins[row, 64 * j + key]) - first_bin
                            lists[row + 32 * half].append([x[row, key], b, counting])
                            if counting:
                                counts[row, b] += 1
            listed = True
        if j & 1 == 0 or not listed or j + 1 >= tiles:
            continue
        listed = False
        most = max(map(len, lists))
        scheduled = j + 1 >= k["FIRST_REFRESH"] and (j + 1) & j == 0
        if most < (min(trig, trig_hard) if scheduled else trig_hard):
            continue
        out["refreshes"] += 1
        for lane, entries in enumerate(lists):
            for e in entries[:k["LIST_CAP"]]:
                if not e[2]:
                    counts[lane & 31, e[1]] += 1
                    e[2] = True
        max_count = max(max_count, int(counts.max()))
        root = np.maximum(_roots(edges, counts, r, h), run - 1.0)
        low = np.maximum(low, root)
        if most > k["LIST_CAP"]:
            break                                            # the block is redone: nothing more is listed
        support = int((counts * (edges[None] > root[:, None])).sum(1).max())
        if (most > k["PRUNE_FROM_COUNTING" if counting else "PRUNE_FROM"] and prunes < k["MAX_PRUNES"] and support <= k["PRUNE_SUPPORT"]
                and support * (1.0 + np.log(tiles / (j + 1))) <= k["PRUNE_SUPPORT_END"]):
            before = sum(map(len, lists))
            lists = [[e for e in entries if e[0] >= low[lane & 31]] for lane, entries in enumerate(lists)]
            prunes += 1
            out["pruned"] += before - sum(map(len, lists))
            out["prunes_leaving_odd_lists"] += any(len(entries) & 1 for entries in lists)
            most = max(map(len, lists))
        out["longest"] = max(out["longest"], most)
        trig = most + k["GROW"]
        tight = most > k["LIST_CAP"] - 3 * k["TILE_ENTRIES"]
        trig_hard = min(most + k["GROW_COUNTING" if counting else "GROW_HARD"], k["LIST_CAP"] + 1)
        if not tight:
            trig_hard = min(trig_hard, k["LIST_CAP"] - 2 * k["TILE_ENTRIES"] + 1)
    out.update(counting=counting, prunes=prunes, max_count=max_count, longest=max(out["longest"], max(map(len, lists))))
    out["overflow"] = out["longest"] > k["LIST_CAP"]
    return out

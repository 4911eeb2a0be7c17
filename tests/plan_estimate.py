"""The planner's estimate of the unit size, in plain Python from its
definition: every size ceil(max_pages / parts) is priced as the busiest
worker's pages and unit costs plus the merge's reads, and the cheapest wins.
Costs in pages * 16.  The queue as it is dealt, for lists and shards too."""
import numpy as np

UNIT, SPLIT, COMBINE = 96, 32, 48


def candidate_parts():
    parts = list(range(1, 65))
    while len(parts) < 96:
        parts.append(parts[-1] + parts[-1] // 8)
    return parts


def unit_size(pages, q_chunk, G, max_partials=1024, unit_cap=1024, listed=False, shard=False):
    """(unit size, units, whether more units than workers go free) for tiles
    of `pages` pages, q_chunk rows a request."""
    P = np.asarray(pages, np.int64)
    longest, best = max(1, int(P.max())), None
    for parts in candidate_parts():
        c = max(1, min(unit_cap, -(-longest // parts)))
        n = -(-P // c)
        W, S = int(n.sum()), int(n.sum() if shard else n[n > 1].sum())
        if S > max_partials or W > len(P) + max_partials:
            continue
        # two whole tiles of at most `pair` pages, their costs included, take
        # no longer than one unit; a tile stands in the queue where its
        # request's longest row puts it (lists: anywhere; past 8,192 tiles the
        # queue is in tile order)
        pair = (16 * c - UNIT - (SPLIT if shard else 0)) / 32
        if q_chunk > 1 and not shard:
            pair = 0 if listed else pair - -(-(q_chunk - 1) // 64)
        if len(P) > 8192:
            pair = 0
        free = G < W and 2 * (W - G) <= int(((P >= 1) & (P <= pair)).sum())
        R = 1 if free else -(-W // G)
        cost = max(R * c * 16 * G, 16 * int(P.sum())) + (R * UNIT + min(R, -(-S // G)) * SPLIT) * G + S * COMBINE
        if best is None or cost < best[0]:
            best = (cost, c, W, free)
    return best[1:]


def busiest(units, G, shard=False):
    """Pages * 16 and unit costs of the busiest worker: slot i of pass k goes to
    worker i, or to G - 1 - i on odd passes (which worker a slot is does not
    matter).  A unit is (tile, first page, last page, partial slot or -1)."""
    loads = np.zeros(G, np.int64)
    for i, u in enumerate(units):
        k, r = divmod(i, G)
        loads[r if k % 2 == 0 else G - 1 - r] += 16 * int(u[2] - u[1]) + UNIT + (SPLIT if shard else 0)
    return loads.max()

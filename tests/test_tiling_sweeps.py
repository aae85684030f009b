"""Index arithmetic of the kernels that take several steps per launch,
replayed on the CPU: the partition of a lattice into a frame of tiles and
sweeping waves (sweep2d.hpp, host_util.hpp), the tiles held in LDS (tile_body,
tile_kernel, ilfbm_tile_kernel).  Every node is one tile's or wave's own, every
load and store lies in the lattice, every LDS read lies in the array and meets
the level it wants; and a planted mistake fails."""
import numpy as np
import pytest

D2Q9 = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1),
        (1, -1)]
DIRS = {3: [(0, 0), (1, 0), (-1, 0)], 5: D2Q9[:5], 9: D2Q9}
SIDE = 16                     # a frame tile's region (kFrameSide)


def sweep_rows(ny):
    return min(32, max(8, (ny // 128 + 3) // 4 * 4))


def sweep_plan(nx, ny, k, rows, px, py, front, frows=0):
    """sweep_plan; front: bit i for a front at wall i (IREBM), frows: rows of
    the segments beside a side wall with a front (0: no such strip)"""
    T = SIDE - 2 * k
    P = dict(k=k, tile=T, xa=0, xb=nx, ya=0, yb=ny, nleft=0, nright=0,
             nside=0, nbottom=0, ntop=0, rows=rows)
    band = [2 if front >> i & 1 else 1 for i in range(4)]
    if not px:
        P.update(nleft=band[0], nright=band[1], nside=-(-ny // T),
                 xa=band[0] * T, xb=nx - band[1] * T)
    if not py:
        P.update(nbottom=band[2], ntop=band[3], ya=band[2] * T,
                 yb=ny - band[3] * T)
    if P["xb"] - P["xa"] < 64 or P["yb"] - P["ya"] < 16:
        return None
    P["nacross"] = -(-(P["xb"] - P["xa"]) // T)
    h = P["yb"] - P["ya"]
    P["frows"] = min(frows, rows) if frows else rows
    P["fl"], P["fr"] = (front & 1, front >> 1 & 1) if frows else (0, 0)
    P["fseg"], P["nseg"] = -(-h // P["frows"]), -(-h // rows)
    return P


def tiles_only(nx, ny):
    """batch_plan where no strip fits"""
    T = SIDE - 8
    return dict(k=4, tile=T, xa=nx, xb=nx, ya=0, yb=ny, nleft=-(-nx // T),
                nright=0, nside=-(-ny // T), nbottom=0, ntop=0, nacross=1,
                rows=1, frows=1, fl=0, fr=0, fseg=0, nseg=0, strips=1)


def cut(P, w):
    strips = P.get("strips") or -(-(P["xb"] - P["xa"]) // w)
    nfl = 1 if P["fl"] and strips > 0 else 0
    nfr = 1 if P["fr"] and strips > nfl else 0
    return strips, nfl, nfr


def frame_tiles(P, nx, ny):
    T, n = P["tile"], P["nleft"] + P["nright"]
    for t in range(n * P["nside"]):
        c, r = t % n, t // n
        left = c < P["nleft"]
        x0 = c * T if left else P["xb"] + (c - P["nleft"]) * T
        yield (x0, min(x0 + T, P["xa"] if left else nx),
               r * ny // P["nside"], (r + 1) * ny // P["nside"])
    w = P["xb"] - P["xa"]
    for t in range((P["nbottom"] + P["ntop"]) * P["nacross"]):
        c, r = t % P["nacross"], t // P["nacross"]
        low = r < P["nbottom"]
        y0 = r * T if low else P["yb"] + (r - P["nbottom"]) * T
        yield (P["xa"] + c * w // P["nacross"],
               P["xa"] + (c + 1) * w // P["nacross"], y0,
               min(y0 + T, P["ya"] if low else ny))


def waves(P, w):
    strips, nfl, nfr = cut(P, w)
    nf, m = nfl + nfr, strips - nfl - nfr
    for k in range(nf * P["fseg"] + m * P["nseg"]):
        if k < nf * P["fseg"]:
            strip = 0 if k % nf < nfl else strips - 1
            rows, y0 = P["frows"], P["ya"] + k // nf * P["frows"]
        else:
            j = k - nf * P["fseg"]
            strip = nfl + j % m
            rows, y0 = P["rows"], P["ya"] + j // m * P["rows"]
        x0 = P["xa"] + strip * w
        yield x0, min(x0 + w, P["xb"]), y0, min(y0 + rows, P["yb"])


def check_wave(x0, x1, y0, y1, K, nx, ny, px, py):
    """lanes and rows that sweep_body loads: they wrap at most once, and on a
    periodic axis only"""
    w = x1 - x0 + 2 * K
    assert x0 < x1 and y0 < y1 and w <= 64
    assert px or (x0 >= K and x1 + K <= nx)
    assert py or (y0 >= K and y1 + K <= ny)
    x = x0 - K + np.minimum(np.arange(64), w - 1)
    x = np.where(x < 0, x + nx, x)
    x = np.where(x >= nx, x - nx, x)
    r = np.arange(y0 - K, y1 + K)
    r = np.where(r < 0, r + ny, np.where(r >= ny, r - ny, r))
    for v, n in ((x, nx), (r, ny)):
        assert v.min() >= 0 and v.max() < n
    # own lanes store own columns
    own = np.arange(64)
    own = own[(own >= K) & (own < w - K)]
    assert np.array_equal(x[own], np.arange(x0, x1))


def check_tile(q, box, k, nx, ny, rx, n, px, py, neu=(0, 0, 0, 0),
               tall=False, hy=None, planted=0):
    """k levels of a tile and its halo: ranges and levels of what it reads.
    planted: levels that the active region fails to shrink by."""
    x0, x1, y0, y1 = box
    hy = k if hy is None else hy
    w, h = x1 - x0 + 2 * k, y1 - y0 + 2 * hy
    t = np.arange(n)
    sx, sy = (n // rx, 1) if tall else (1, rx)
    lx, ly = (t // sx, t % sx) if tall else (t % sy, t // sy)
    assert w <= rx and w * h <= n and h <= n // rx
    x, y = x0 - k + lx, y0 - hy + ly
    gx, gy = (x % nx if px else x), (y % ny if py else y)
    node = (lx < w) & (ly < h) & (gx >= 0) & (gx < nx) & (gy >= 0) & (gy < ny)
    own = node & (x >= x0) & (x < x1) & (y >= y0) & (y < y1)
    assert own.sum() == (x1 - x0) * (y1 - y0)
    mx, my = gx.copy(), gy.copy()
    for i, (a, at, to) in enumerate(((0, 0, 1), (0, nx - 1, nx - 2),
                                     (1, 0, 1), (1, ny - 1, ny - 2))):
        if neu[i]:
            m = (gx if a == 0 else gy) == at
            (mx if a == 0 else my)[m] = to
    mirror = node & ((mx != gx) | (my != gy))
    mt = t + (mx - gx) * sx + (my - gy) * sy
    level = np.where(node, 0, -1)
    for m in range(1, k + 1):
        s = max(m - planted, 0)
        act = node & (lx >= s) & (lx < w - s)
        if q != 3:
            act &= (ly >= s) & (ly < h - s)
        assert act[own].all()
        for ex, ey in DIRS[q]:
            src = t - ex * sx - ey * sy
            assert src[act].min() >= 0 and src[act].max() < n
            known = act.copy()
            if not px:
                known &= (gx - ex >= 0) & (gx - ex < nx)
            if not py:
                known &= (gy - ey >= 0) & (gy - ey < ny)
            assert (level[src[known]] == m - 1).all()
            at = act & mirror
            if at.any():
                src = mt - ex * sx - ey * sy
                assert src[at].min() >= 0 and src[at].max() < n
                assert (level[src[at]] == m - 1).all()
        level[act] = m
    assert (level[own] == k).all()


def covered(boxes, nx, ny):
    seen = np.zeros((ny, nx), int)
    for x0, x1, y0, y1 in boxes:
        assert 0 <= x0 < x1 <= nx and 0 <= y0 < y1 <= ny
        seen[y0:y1, x0:x1] += 1
    assert (seen == 1).all()


SIZES = [(88, 40), (89, 33), (120, 560), (1700, 32), (64, 77), (145, 431),
         (257, 251), (88, 300)]


@pytest.mark.parametrize("nx,ny", SIZES)
@pytest.mark.parametrize("px,py", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("front", [0, 1, 2, 4, 15])
def test_sweep_partition(nx, ny, px, py, front):
    if px:
        front &= 12
    if py:
        front &= 3
    found = False
    for plan_k, rows, frows in ((4, sweep_rows(ny), 0), (4, 32, 2),
                                (3, 16, 2), (4, 32, 8)):
        P = sweep_plan(nx, ny, plan_k, rows, px, py, front, frows)
        if P is None:
            continue
        found = True
        tiles = list(frame_tiles(P, nx, ny))
        for K in range(1, plan_k + 1):
            # a single lattice cuts its strips for K, a batch for the plan's
            for w in {64 - 2 * K, 64 - 2 * plan_k}:
                ws = list(waves(P, w))
                covered(tiles + ws, nx, ny)
                for b in ws:
                    check_wave(*b, K, nx, ny, px, py)
        ns = (P["nleft"] + P["nright"]) * P["nside"]
        for i in {0, ns - 1, ns, len(tiles) - 1} & set(range(len(tiles))):
            for K in range(1, plan_k + 1):
                neu = (0, 0, 0, 0) if px or py else (0, 1, 0, 1)
                check_tile(9, tiles[i], K, nx, ny, SIDE, SIDE * SIDE, px, py,
                           neu, tall=i < ns)
    if not px and not py and (nx, ny) == (88, 40):
        assert found == (front in (0, 1, 2, 4))


@pytest.mark.parametrize("nx,ny", [(3, 3), (5, 40), (63, 9), (70, 15)])
@pytest.mark.parametrize("px", [0, 1])
def test_batch_lattices_of_tiles_alone(nx, ny, px):
    P = tiles_only(nx, ny)
    tiles = list(frame_tiles(P, nx, ny))
    covered(tiles, nx, ny)
    assert not list(waves(P, 56))
    for b in tiles:
        for K in range(1, 5):
            check_tile(9, b, K, nx, ny, SIDE, SIDE * SIDE, px, px, tall=True)


def tile_plan(q, eebm, nx, ny):
    n = nx * ny
    if n > 60000 and min(nx, ny) < 64:
        k, side = ((4, 14) if eebm and n <= (200000 if nx < 64 else 100000)
                   else (0, 0))
    elif eebm:
        k, side = ((6, 8) if n <= 15000 else (4, 8) if n <= 60000 else
                   (0, 0))
    else:
        k, side = ((4, 8) if n <= 30000 else (3, 10) if n <= 110000 else
                   (2, 12) if n <= 130000 else (0, 0))
    if not k:
        return None
    ntx, nty = -(-nx // side), -(-ny // side)
    return k, ntx, nty, -(-nx // ntx) + 2 * k, -(-ny // nty) + 2 * k


@pytest.mark.parametrize("nx,ny", [(3, 3), (4, 3), (9, 8), (17, 3), (8, 25),
                                   (40, 33), (173, 173), (331, 331),
                                   (57, 1136), (5000, 20)])
@pytest.mark.parametrize("eebm", [False, True])
def test_tile_kernel(nx, ny, eebm):
    plan = tile_plan(9, eebm, nx, ny)
    if nx * ny > 60000 and eebm == (nx == ny):
        assert plan is None
        return
    k, ntx, nty, rx, ry = plan
    assert rx * ry <= 1024 and rx * ry * 9 * 8 <= 65536
    boxes = [(c * nx // ntx, (c + 1) * nx // ntx, r * ny // nty,
              (r + 1) * ny // nty) for r in range(nty) for c in range(ntx)]
    covered(boxes, nx, ny)
    some = boxes if len(boxes) < 30 else boxes[:2] + boxes[-2:] + \
        [boxes[ntx - 1], boxes[-ntx]]
    for b in some:
        for K in range(1, k + 1):
            for px, py, neu in ((0, 0, (1, 1, 1, 1)), (1, 1, (0,) * 4),
                                (0, 1, (0, 1, 0, 0))):
                check_tile(9, b, K, nx, ny, rx, rx * ry, px, py, neu)


@pytest.mark.parametrize("q,nx,ny", [(9, 3, 3), (9, 16, 8), (9, 17, 9),
                                     (5, 33, 40), (9, 100, 17), (3, 513, 1),
                                     (3, 2100, 1), (9, 61, 62)])
def test_ilfbm_tiles(q, nx, ny):
    """blocks of 1024 threads, 32 x 32 in 2D, for launches of 1 to 8
    iterations"""
    rx = 1024 if q == 3 else 32
    for kk in range(1, 9):
        ntx = -(-nx // (rx - 2 * kk))
        nty = 1 if q == 3 else -(-ny // (32 - 2 * kk))
        boxes = [(c * nx // ntx, (c + 1) * nx // ntx, r * ny // nty,
                  (r + 1) * ny // nty) for r in range(nty)
                 for c in range(ntx)]
        covered(boxes, nx, ny)
        for b in boxes[:3] + boxes[-2:]:
            for px, py, neu in ((0, 0, (1, 1, 1, 1)), (1, 1, (0,) * 4)):
                if q == 3:
                    py, neu = 1, (neu[0], neu[1], 0, 0)
                check_tile(q, b, kk, nx, ny, rx, 1024, px, py, neu,
                           hy=0 if q == 3 else kk)


def test_planted_mistakes_are_seen():
    box = (16, 24, 16, 24)
    check_tile(9, box, 4, 200, 200, SIDE, SIDE * SIDE, 0, 0)
    with pytest.raises(AssertionError):   # a region that does not shrink
        check_tile(9, box, 4, 200, 200, SIDE, SIDE * SIDE, 0, 0, planted=1)
    with pytest.raises(AssertionError):   # a tile too wide for its halo
        check_tile(9, (16, 25, 16, 24), 4, 200, 200, SIDE, SIDE * SIDE, 0, 0)
    with pytest.raises(AssertionError):   # a Neumann wall tile one node wide
        check_tile(9, (199, 200, 16, 24), 4, 200, 200, SIDE, SIDE * SIDE, 0,
                   0, (0, 1, 0, 0))
    P = sweep_plan(300, 200, 4, 16, 0, 0, 1, 2)
    P["fseg"] -= 1
    with pytest.raises(AssertionError):   # a segment left out
        covered(list(frame_tiles(P, 300, 200)) + list(waves(P, 56)), 300, 200)
    with pytest.raises(AssertionError):   # a strip too wide for a wave
        check_wave(20, 80, 20, 36, 4, 300, 200, 0, 0)
    with pytest.raises(AssertionError):   # a segment at a wall with no frame
        check_wave(20, 76, 182, 198, 4, 300, 200, 1, 0)

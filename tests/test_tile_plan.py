"""The row counts that test_gpu_predictor_bf16.py runs through the tiles of the maps of all rows: here, with a copy of the rule
that picks the tiles, that together they reach every kind of tile there is."""
import numpy as np

HEIGHTS, COSTS = (8, 7, 6, 5, 4), (1000, 888, 780, 690, 600)      # tile heights in blocks of 32 rows; thousandths of a round
KEY_SLACK, ROW_ALIGN, ROW_TILE = 64, 8, 256
# of a model of hidden size 256 and 3072 feed-forward units: (tile columns, rows beyond the activations')
MAPS = {"query-key-value": (3, KEY_SLACK), "key-value": (2, KEY_SLACK), "back to hidden": (1, 0), "feed-forward": (12, 0)}
ROWS = [2624, 2696, 2728, 3464, 10760, 13672, 16072, 19080, 24264, 24744, 32456, 32872, 36008, 41096, 43912, 49160, 50856,
        65480, 65704, 73816, 78248, 148120]


def plan(rows, columns):
    """(256-row tiles in front, height of the others): the cheapest of 15 ways to cut a map's rows for 256 workgroups."""
    tiles, ways = -(-rows // 256) * columns, []
    for lane in range(15):
        h, c, pick = HEIGHTS[lane % 5], COSTS[lane % 5], lane // 5
        rounds = max(0 if pick == 0 else tiles // 256 - (pick - 1), 0)
        front = rounds * 256 // columns
        rest = -(-max(rows - 256 * front, 0) // (32 * h)) * columns
        cost = rounds * 1000 + rest // 256 * c + (50 if rounds > 0 else 0)
        if rounds == 0 and rest <= 256:
            cost = c
        elif rest % 256:
            cost += c * max(680, rest % 256 * 1000 // 256) // 1000
        ways.append((cost, lane, front, h))
    return min(ways)[2:]


def lengths_of(rows, rng):
    """Requests, a multiple of 20, that fill `rows` rows of the activations and leave the fewest rows behind them: every length
    is one more than a multiple of 8, so that nothing of the workspace's allowance for alignment is left over."""
    units = rows // ROW_ALIGN
    n = 20 * -(-units // (20 * 72))
    u = np.full(n, units // n)
    u[:units % n] += 1
    shift = rng.integers(-4, 5, n // 2)
    u[:n // 2] += shift
    u[n // 2:2 * (n // 2)] -= shift
    return (u * ROW_ALIGN - 7).astype(np.int32)


def kinds(rows):
    """What the maps of a call of lengths_of(rows) meet: (map, tiles behind whole rounds, height, last one past the buffers)."""
    max_rows = -(-(rows + KEY_SLACK) // ROW_TILE) * ROW_TILE
    met = set()
    for name, (columns, extra) in MAPS.items():
        if max_rows // 256 * columns < 128:                      # tiles of 128 rows, no plan
            continue
        front, h = plan(rows + extra, columns)
        left = rows + extra - 256 * front
        if left > 0:
            met.add((name, front > 0, 32 * h, 256 * front - (-left // (32 * h)) * 32 * h > max_rows))
    return met


def test_row_counts_reach_every_kind_of_tile():
    met = set().union(*[kinds(r) for r in ROWS])
    for name in MAPS:
        for height in (256, 224, 192, 160, 128):
            assert (name, False, height, False) in met, (name, height)
        for height in (224, 192, 160):                           # (the buffers end on whole tiles of 256 and 128 rows)
            assert (name, False, height, True) in met, (name, height)
        assert any((name, True, height, True) in met for height in (224, 192, 160)), name
    for rows in ROWS:
        lengths = lengths_of(rows, np.random.default_rng(rows))
        assert (lengths % 8 == 1).all() and lengths.min() > 0 and lengths.max() <= 640
        assert int((lengths + 7).sum()) == rows

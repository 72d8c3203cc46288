"""The library's tile choice in Python, read from the table in its source, so that a refitted table does not silently move a shape to
another tile; and model shapes whose two branch layers (attention projection: rows x hidden x hidden, second MLP layer: rows x hidden x
mlp_hidden) fall on each tile that the library runs the branch epilogue on."""
import math
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COMPUTE_UNITS = 256

# rows, grid (tokens = grid^2), hidden, heads, mlp_hidden, (tile of the projection, tile of the second MLP layer)
# tokens divide no tile height, so tiles span rows of the batch; hidden is no multiple of most tile widths
CASES = [
    (6, 15, 360, 5, 424, ((64, 64), (64, 64))),
    (12, 15, 360, 5, 1288, ((128, 64), (128, 64))),
    (7, 17, 1440, 20, 5760, ((128, 64), (128, 128))),
    (56, 14, 360, 5, 424, ((128, 128), (128, 128))),
    (55, 20, 360, 5, 424, ((128, 192), (128, 192))),
    (11, 15, 792, 11, 3168, ((64, 64), (96, 128))),
    (33, 20, 792, 11, 640, ((128, 128), (256, 256))),
    (35, 9, 1440, 20, 5760, ((128, 128), (192, 128))),
    (24, 15, 768, 12, 3072, ((128, 128), (256, 128))),
]

# the same with tiles inside one row of the batch: every tile of the largest kind (residual half a tile at a time, planes token by token), and
# some of the 256- and 192-row tiles that find the residual a whole tile ahead (row heights up to 128 have such tiles above)
INSIDE_ROWS = [(16, 32, 1024, 16, 1024, ((256, 256), (256, 256))),
               (14, 17, 1440, 20, 5760, ((128, 128), (256, 128))),
               (5, 24, 1440, 20, 5760, ((128, 128), (192, 128)))]

# rows, features, K and activation of layers that only store, all of them on the largest tile
LARGEST = [(4089, 4092, 64, 1), (4089, 4092, 128, 0), (4089, 4088, 192, 1), (4096, 4096, 256, 2), (3841, 3844, 320, 0)]

# rows, features and K of layers that only store: every tile, ragged rows and columns, tails of K where the tile takes them, and
# 256x128 (three stages, two groups of loaders) at 3 n, 3 n + 1 and 3 n + 2 K-steps
STORES = [(1, 16, 8), (33, 4, 128), (65, 140, 200), (3401, 264, 8), (257, 3304, 136), (771, 2500, 136), (1034, 3592, 384), (132, 3408, 328), (1715, 3524, 248),
          (3839, 3224, 456), (2461, 3280, 456), (2348, 2528, 512), (3588, 4000, 64), (3437, 3460, 520), (845, 3076, 6152), (500, 3076, 3080), (3603, 796, 1912),
          (7359, 772, 768), (7177, 784, 832), (7277, 772, 896), (3209, 2520, 880), (741, 3424, 40)]


def _source():
    return open(os.path.join(ROOT, "paper_2509_11628_amd", "csrc", "gemm_mfma.hip")).read()


def tile_table():
    src = _source()
    body = src[src.index("kTileKinds[] = {"):]
    body = body[:body.index("};")]
    rows = re.findall(r"\{(\d+), (\d+), ([\d.]+)f, ([\d.]+)f, ([\d.]+)f, ([\d.]+)f, ([\d.]+)f, ([\d.]+)f, (\w+), (\w+)\}", body)
    return [tuple(int(v) for v in r[:2]) + tuple(float(v) for v in r[2:8]) + tuple(v == "true" for v in r[8:]) for r in rows]


def branch_tile(table, M, N, K):
    """(height, width) of the tile for a layer with the branch epilogue, and how much dearer the next best one is modelled."""
    costs = []
    for bm, bn, a, _, b, _, cb, rb, two, whole_steps in table:
        if cb == 0.0 or (whole_steps and (K % 64 or K < 64)):
            continue
        depth = math.ceil(math.ceil(M / bm) * math.ceil(N / bn) / COMPUTE_UNITS)
        odd = depth % 2
        rounds = (depth - odd) / 2 * (1.0 + rb) + odd if two else 1.0 + rb * (depth - 1)
        costs.append((a + (cb + b * math.ceil(K / 64)) * rounds, (bm, bn)))
    costs.sort()
    return costs[0][1], costs[1][0] / costs[0][0]


def _store_cost(kind, M, N, K):
    bm, bn, a, c, b, r, _, _, two, _ = kind
    depth = math.ceil(math.ceil(M / bm) * math.ceil(N / bn) / COMPUTE_UNITS)
    odd = depth % 2
    return a + (c + b * math.ceil(K / 64)) * ((depth - odd) / 2 * (1.0 + r) + odd if two else 1.0 + r * (depth - 1))


def store_kind(table, M, N, K):
    """Place in the table of the cheapest tile for a layer that only stores, its modelled time and that of the next one."""
    costs = sorted((_store_cost(k, M, N, K), i) for i, k in enumerate(table) if not k[9] or K % 64 == 0)
    return costs[0][1], costs[0][0], costs[1][0]


def store_tile(table, M, N, K):
    """(height, width) of the tile for a layer that only stores, the columns that run on the largest tile ahead of it in a launch of
    their own, and how much dearer the next best single tile is modelled."""
    second = float(re.search(r"kSecondLaunch = ([\d.]+);", _source()).group(1))
    kind, cost, runner_up = store_kind(table, M, N, K)
    head, margin = 0, runner_up / cost
    if M >= 256 and K % 64 == 0:
        rounds = 1
        while (n1 := rounds * COMPUTE_UNITS // math.ceil(M / 256) * 256) < N:
            rounds += 1
            if n1 < 256:
                continue
            tail, rest, _ = store_kind(table, M, N - n1, K)
            rest += _store_cost(table[0], M, n1, K)
            if rest < cost if head else rest + second < 0.96 * cost:
                kind, head, cost = tail, n1, rest
    return table[kind][:2], head, margin

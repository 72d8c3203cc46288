"""The library's tile choice in Python, read from the table in its source, so that a refitted table does not silently move a shape to
another tile; and model shapes whose two branch layers (attention projection: rows x hidden x hidden, second MLP layer: rows x hidden x
mlp_hidden) fall on each tile that the library runs the branch epilogue on."""
import math
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COMPUTE_UNITS = 256

# rows, grid (tokens = grid^2), hidden, heads, mlp_hidden, (kind of the projection, kind of the second MLP layer: places in the table)
# tokens divide no tile height, so tiles span rows of the batch; hidden is no multiple of most tile widths
CASES = [
    (6, 15, 360, 5, 424, (5, 5)),
    (12, 15, 360, 5, 1288, (4, 4)),
    (7, 17, 1440, 20, 5760, (2, 12)),
    (56, 14, 360, 5, 424, (8, 8)),
    (55, 20, 360, 5, 424, (8, 8)),
    (11, 15, 792, 11, 3168, (5, 5)),
    (33, 20, 792, 11, 640, (3, 13)),
    (35, 9, 1440, 20, 5760, (3, 13)),
    (24, 15, 768, 12, 3072, (11, 13)),
    (12, 15, 360, 5, 640, (4, 11)),
    (17, 12, 792, 11, 640, (5, 12)),
    (28, 14, 360, 5, 3168, (2, 10)),
    (38, 17, 360, 5, 3168, (8, 7)),
    (24, 17, 792, 11, 640, (3, 1)),
    (49, 17, 792, 11, 640, (3, 0)),
]

# the same with tiles inside one row of the batch: every tile of the largest kind (residual half a tile at a time, planes token by token), and
# some of the 256- and 192-row tiles that find the residual a whole tile ahead (row heights up to 128 have such tiles above)
INSIDE_ROWS = [(16, 32, 1024, 16, 1024, (0, 0)),
               (14, 17, 1440, 20, 5760, (3, 1)),
               (5, 24, 1440, 20, 5760, (3, 13))]

# rows, features, K and activation of layers that only store, all of them on the largest tile
LARGEST = [(4089, 4092, 64, 1), (4089, 4092, 128, 0), (4089, 4088, 192, 1), (4096, 4096, 256, 2), (3841, 3844, 320, 0)]

# rows, features and K of layers that only store: every kind, ragged rows and columns, tails of K where the kind takes them, and the tiles of
# two wave groups (places 1, 11, 12, 13) at one to six and at 3 n, 3 n + 1 and 3 n + 2 K-steps, fewer and more than the ring has stages
STORES = [(1, 16, 8), (33, 4, 128), (65, 140, 200), (3401, 264, 8), (257, 3304, 136), (771, 2500, 136), (1034, 3592, 384), (132, 3408, 328), (1715, 3524, 248),
          (3839, 3224, 456), (2461, 3280, 456), (2348, 2528, 512), (3588, 4000, 64), (3437, 3460, 520), (845, 3076, 6152), (500, 3076, 3080), (3603, 796, 1912),
          (7359, 772, 768), (7177, 784, 832), (7277, 772, 896), (3209, 2520, 880), (741, 3424, 40),
          (4889, 3100, 320), (4916, 3180, 256), (5889, 2620, 384), (31, 4, 64), (5506, 132, 128), (5444, 136, 192), (5567, 132, 256), (5713, 136, 320),
          (5647, 284, 64), (5468, 280, 128), (5460, 336, 192), (518, 3604, 256), (513, 3636, 320), (6055, 648, 192), (1697, 2308, 256), (5525, 652, 320),
          (5498, 652, 384), (5398, 1096, 40), (5941, 2564, 64), (4995, 1540, 384)]

# fp32 models: rows, grid, hidden, heads, mlp_hidden, (kernels of the two branch layers, as launch_gemm_f32 counts them: 5 .. 8 are the tiles
# through LDS).  A row alone runs straight from memory.
F32_CASES = [(30, 13, 192, 3, 576, (5, 5)), (12, 13, 320, 5, 640, (6, 6)), (9, 11, 384, 6, 1536, (7, 7)), (7, 9, 384, 6, 1536, (8, 8)), (25, 9, 64, 4, 128, (8, 8))]

# rows, text tokens, latent height and width (patch 2), hidden, heads, mlp_hidden, kinds (places in the table) of the launches for both streams:
# qkv, projection, first MLP layer, second one, second one where it is verified.  Streams shorter than a tile, that end inside tiles and tiles that
# span rows of the batch; a row alone takes 64x128.
STREAM_LAYERS = ("qkv", "proj", "fc1", "fc2", "truth")
STREAMS = [(64, 17, 46, 66, 256, 4, 64, (0, 0, 1, 0, 0)), (64, 40, 68, 44, 128, 2, 256, (0, 1, 0, 1, 1)), (13, 129, 40, 60, 768, 12, 768, (1, 1, 1, 1, 1)),
           (64, 5, 38, 28, 128, 2, 64, (12, 12, 12, 12, 12)), (48, 40, 32, 52, 256, 4, 64, (13, 13, 12, 11, 13)), (64, 77, 38, 46, 128, 2, 64, (1, 11, 13, 11, 13)),
           (9, 77, 60, 58, 512, 8, 1024, (0, 13, 0, 13, 13)), (2, 1, 16, 16, 128, 2, 512, (11, 11, 11, 11, 11))]


def _source():
    return open(os.path.join(ROOT, "paper_2509_11628_amd", "csrc", "gemm_mfma.hip")).read()


def tile_table():
    src = _source()
    body = src[src.index("kTileKinds[] = {"):]
    body = body[:body.index("};")]
    rows = re.findall(r"\{(\d+), (\d+), ([\d.]+)f, ([\d.]+)f, ([\d.]+)f, ([\d.]+)f, ([\d.]+)f, ([\d.]+)f, (\w+), (\w+)\}", body)
    return [tuple(int(v) for v in r[:2]) + tuple(float(v) for v in r[2:8]) + tuple(v == "true" for v in r[8:]) for r in rows]


def branch_tile(table, M, N, K):
    """Place in the table of the tile for a layer with the branch epilogue, and how much dearer the next best one is modelled."""
    costs = []
    for place, (bm, bn, a, _, b, _, cb, rb, two, whole_steps) in enumerate(table):
        if cb == 0.0 or (whole_steps and (K % 64 or K < 64)):
            continue
        depth = math.ceil(math.ceil(M / bm) * math.ceil(N / bn) / COMPUTE_UNITS)
        odd = depth % 2
        rounds = (depth - odd) / 2 * (1.0 + rb) + odd if two else 1.0 + rb * (depth - 1)
        costs.append((a + (cb + b * math.ceil(K / 64)) * rounds, place))
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

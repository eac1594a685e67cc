"""Words that the plan part of an attention workspace may hold where no plan was built, for calls
that take ranges of equal cost (fewer than 512 units, no given split): the number of ranges and one
record of eight words per cut (request, row block, tile, first row, rows, keys, two unused)."""
import numpy as np

INT_MAX = 0x7FFFFFFF
EXTREMES = np.array([-2**31, -2**31 + 1, -65536, -16, -1, 0, 1, 2, 3, 15, 16, 17, 63, 64, 65, 1000, 65536, 1 << 22,
                     INT_MAX - 16, INT_MAX - 1, INT_MAX], np.int64)

# (Hq, Hkv, d, page, b, contexts); the last one has a single range and a single unit
SHAPES = [
    (16, 4, 128, 64, 8, (700, 64, 1200, 3, 65)),
    (32, 2, 64, 16, 16, (500, 2100, 40)),
    (64, 4, 128, 64, 16, (900, 3000, 130)),      # whole-tile waves
    (12, 1, 128, 4, 4, (40,)),
]
KINDS = ["bytes 00", "bytes 01", "bytes 7f", "bytes ff", "negative count", "rows at 2^31", "keys at 2^31",
         "stray tiles"] + [f"mix {s}" for s in range(6)]


def ranges_of(Hq, Hkv, b, R, max_kv_len):
    """Most ranges per kv-head (the layout of the library's workspace)."""
    rows = Hq // Hkv * b
    blocks = -(-rows // (256 if rows > 128 else 128))
    per_head = 256 // Hkv
    assert per_head * Hkv * 10 >= 256 * 9
    return min(per_head, R * blocks * -(-max_kv_len // 64))


def words(kind, ranges, R, b, qo, kv_lens):
    """(count, records) as int32"""
    rec = np.zeros((ranges + 1, 8), np.int64)
    count = ranges
    i = np.arange(ranges + 1)
    if kind.startswith("bytes"):
        w = int(kind[6:] * 4, 16)
        rec[:] = w
        count = w
    elif kind == "negative count":  # the bits of -3.0f
        rec[:] = 0xC0400000
        count = 0xC0400000
    elif kind in ("rows at 2^31", "keys at 2^31"):
        rec[:, 0] = i * R // (ranges + 1)
        rec[:, 2] = i % 2
        rec[:, 4], rec[:, 5] = 1, 100
        if kind.startswith("rows"):
            rec[:, 3] = INT_MAX
        else:
            rec[:, 5] = np.where(i % 2 == 0, INT_MAX, -2**31)
    elif kind == "stray tiles":  # a plan's own packing, cut where no plan cuts
        r = i * R // ranges
        rec[:, 0] = r
        rec[:, 2] = np.where(r < R, 1 + i % 2, 0)
        rr = np.minimum(r, R - 1)
        rec[:, 3], rec[:, 4], rec[:, 5] = qo[rr], qo[rr + 1] - qo[rr], kv_lens[rr]
    else:
        g = np.random.default_rng(int(kind.split()[1]))
        near = np.array([R, 2, 8, int(qo[-1]), b, int(np.max(kv_lens)), 1, 1])
        rec = g.integers(-1, 2 * near + 1, size=rec.shape)
        wild = g.random(rec.shape) < 0.15
        rec[wild] = g.choice(EXTREMES, size=int(wild.sum()))
        count = ranges + int(g.integers(-3, 1000))
    as32 = lambda x: (np.asarray(x, np.int64) & 0xFFFFFFFF).astype(np.uint32).view(np.int32)  # noqa: E731
    return int(as32([count])[0]), np.ascontiguousarray(as32(rec))


def case(shape):
    """(block depths, packing, key counts) of a shape"""
    Hq, Hkv, d, page, b, ctx = shape
    k = np.array([b - j % b for j in range(len(ctx))], np.int32)
    qo = np.concatenate([[0], np.cumsum(k)]).astype(np.int32)
    return k, qo, (np.array(ctx) + k).astype(np.int32)

"""Which tile height the large bf16 products take (test helper): k_gemm.hip's phase_rows in Python, so that a test states
the height that it is about.  n_tiles: columns over 128 (gate/up and its backward) or 256 (the others)."""


def phase_rows(M, n_tiles):
    def tiles(bm):
        return -(-M // bm) * n_tiles

    def cost(bm, w):
        return -(-tiles(bm) // 256) * w
    best, c = 256, cost(256, 125)
    if tiles(192) <= 8 * 256 and cost(192, 100) < c:
        best, c = 192, cost(192, 100)
    if tiles(128) <= 4 * 256 and cost(128, 75) < c:
        best = 128
    return best

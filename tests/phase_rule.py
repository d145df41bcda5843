"""Which tile height the large bf16 products take (test helper): k_gemm.hip's phase_rows in Python, so that a test states
the height that it is about.  n_tiles: columns over 128 (gate/up and its backward) or 256 (the others); spill: the
products whose 256-row epilogue spills (the gate/up backward and the router backward's dL/dhbar)."""


def phase_rows(M, n_tiles, spill=False):
    def tiles(bm):
        return -(-M // bm) * n_tiles

    def cost(bm, w):
        return -(-tiles(bm) // 256) * w
    best, c = 256, cost(256, 152 if spill else 125)
    if (spill or tiles(192) <= 8 * 256) and cost(192, 100) < c:
        best, c = 192, cost(192, 100)
    if tiles(128) <= 4 * 256 and cost(128, 80 if spill else 75) < c:
        best = 128
    return best

"""The library's rules for which kernel an output tile runs in (as documented
in include/lors.h), restated for the tests: forwards of few tokens have a
kernel of their own; elsewhere a short last wave of 256 x 256 tiles is cut into
thin tiles, or, on shapes without whole tiles and with LORS_FLAG_SPLIT_LAST_WAVE,
over K -- which shapes split, into how many pieces, and which output tiles run
in pieces."""


def up256(n):
    return -(-n // 256) * 256


def split_budget(R, C, r):
    """Bytes the split partials may use: the workspace (transposed mask,
    padded copy of B, partials) stays below R*C/4."""
    mt = up256(C * -(-R // 32) * 4)
    bpad = up256(2 * R * (-(-r // 8) * 8)) if r % 8 else 0
    return max(0, R * C // 4 - mt - bpad - 256)


def pieces(tiles, nk, budget, cus=256):
    """Pieces per tile of the short last wave (1: no split)."""
    tail = tiles % cus
    if tail == 0 or 2 * tail > cus:
        return 1
    s = min(8, cus // tail, nk // 4, budget // (tail * 256 * 256 * 4))
    return s if s >= 2 else 1


def split_bytes(tiles, nk, budget, cus=256):
    s = pieces(tiles, nk, budget, cus)
    return (tiles % cus) * s * 256 * 256 * 4 if s > 1 else 0


def fwd_group_rows(tiles_m, tiles_n):
    """Tile rows the forward walks at a time (dX: always 4)."""
    return 8 if tiles_m * tiles_n > 256 and tiles_m <= 32 else 4


def split_tiles(rows, cols, cus=256, group_m=4):
    """(row0, col0) of the output tiles that run in pieces, given that the
    grid splits: the logical tiles past the whole waves, mapped to tiles in
    the kernels' grouped order (group_m tile rows at a time, column-major
    inside a group)."""
    tm_n, tn_n = -(-rows // 256), -(-cols // 256)
    tiles = tm_n * tn_n
    out = []
    for t in range(tiles - tiles % cus, tiles):
        per_group = group_m * tn_n
        g = t // per_group
        first = g * group_m
        gsz = min(tm_n - first, group_m)
        within = t - g * per_group
        out.append((256 * (first + within % gsz), 256 * (within // gsz)))
    return out


def few_tokens(L, R, C, cus=256):
    """The forward's kernel for few tokens, which never splits: at most 32
    tokens, or at most one 64-token, 32-feature workgroup per CU."""
    return C <= 1 << 24 and (L <= 32 or -(-R // 32) * -(-L // 64) <= cus)


def fwd_whole_tiles(L, R, C):
    """The forward's fixed-offset copies: whole 256 x 256 tiles over L x R,
    64-wide K-steps over C, 256 slab rows of C bf16 addressed in 32 bits."""
    return L % 256 == 0 and R % 256 == 0 and C % 64 == 0 and 256 * C * 2 < 2**31


def dx_whole_tiles(L, R, C):
    """The same for dX: tiles over L x C, K-steps over R."""
    return L % 256 == 0 and C % 256 == 0 and R % 64 == 0 and 256 * R * 2 < 2**31 and 64 * C * 2 < 2**31


def thin_grid(L, N, cus=256):
    """Tokens per thin tile of a grid that is one short wave: the least of
    rounds x cost of a K-step, the larger tile on a tie."""
    cost = lambda tm: -(-(-(-L // tm) * -(-N // 128)) // cus) * (0.45 + 0.0042 * tm)  # noqa: E731
    return min((256, 192, 128, 64), key=cost)


def kernels(kind, L, R, C, r, cus=256):
    """The kernels that a call without the split flag runs ("few", "whole", or
    the tokens per thin tile), and whether they check every lane of a copy."""
    if kind == "fwd" and few_tokens(L, R, C, cus):
        return {"few"}, C % 64 != 0
    N, K = (R, C) if kind == "fwd" else (C, R)
    checked = K % 64 != 0 or 256 * K * 2 >= 2**31 or (kind == "dx" and 64 * C * 2 >= 2**31)
    tiles = -(-L // 256) * -(-N // 256)
    if r <= 64:
        tail = tiles % cus
        if tail == 0 or 2 * tail > cus:
            return {"whole"}, checked
        if tail == tiles:
            return {thin_grid(L, N, cus)}, checked
        return {"whole", 512 // thin_q(tiles, cus)}, checked
    if 2 * tiles <= cus:  # above rank 64: feature halves only
        return {thin_grid(L, N, cus)}, checked
    rest = (2 * tiles % cus + 1) // 2
    return ({256, 64 if 8 * rest <= cus else 128} if 0 < 4 * rest <= cus else {256}), checked


def thin_q(tiles, cus=256):
    """Thin tiles per tile of the short last wave (1: not cut): the largest
    of 2, 4, 8 whose thin tiles fit on the CUs."""
    tail = tiles % cus
    if tail == 0 or 2 * tail > cus:
        return 1
    q = 2
    while q < 8 and 2 * q * tail <= cus:
        q *= 2
    return q

"""Into how many parts an fp32 layer cuts its GEMM2 tiles, as the library decides it (tests of a number of parts make sure that they run it)."""
from __future__ import annotations

BM, BN, MAX_PARTS, MAX_TILES, CUS = 128, 64, 8, 128, 256


def most_tiles(T, d, E, k):
    """GEMM2 tiles a layer can have, whatever its load."""
    return (T * k // BM + min(T * k, E)) * -(-d // BN)


def parts(T, d, E, k, f):
    avg = T * k // E
    tiles = min(T * k, E) * (avg // BM + 1) * -(-d // BN)  # that are likely
    length = f * max(32, min(avg, BM) + 16) // 32
    if most_tiles(T, d, E, k) > MAX_TILES or length < 768:
        return 1
    return max(1, min(CUS // tiles, MAX_PARTS, f // 128, length // (256 if tiles <= 32 else 512 if tiles <= 64 else 768)))


def workspace_growth(T, d, E, k, f, capacity=0):
    """Bytes by which the workspace of a layer exceeds that of the same layer with f = 16, which cuts nothing."""
    def up(n):
        return -(-n // 256) * 256
    N, nt2, S = T * k, -(-d // BN), parts(T, d, E, k, f)
    rows = E * capacity if capacity else N
    blocks = N // BM + 2 * E  # a ready queue holds these, times the column tiles and their parts, and a combine task per token
    growth = up(rows * f * 4) - up(rows * 16 * 4) + up(32 * (blocks * nt2 * S + T)) - up(32 * (blocks * nt2 + T))
    if S > 1:
        tiles = most_tiles(T, d, E, k)
        growth += up(tiles * 128) + up(tiles * S * min(N, BM) * BN * 4)
    return growth


def combine_tasks(T, R):
    """Combine tasks under the ready-queue scheduler: equal shares of every destination's tokens where twice as many tasks make them equal."""
    per_dest, want = T // R, -(-(T // R) // -(-T // CUS))
    return R * next((n for n in range(want, min(2 * want, per_dest) + 1) if per_dest % n == 0), want)

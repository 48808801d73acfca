"""Which form of the bf16 gate a problem takes, as the library decides it (tests of one form make sure that they run it)."""
from __future__ import annotations

MAX_EXPERTS, CUS = 256, 256


def direct_tokens(T):
    """Tokens of a task of the direct gate (exact logits of all experts, a task per CU)."""
    return 1 if T <= 256 else 2 if T <= 512 else 4


def is_direct(T, E, d, alone):
    """alone: moe_route; else the gate inside the layer."""
    if T <= 256 or (T <= 512 and E <= 128):
        most = 1 << 20
    else:
        most = 1 << 19 if T <= 512 or alone else 1 << 16
    return E % 8 == 0 and T <= 1024 and direct_tokens(T) * d * 4 <= 96 * 1024 and E * d <= most


def direct_sums_alone(T, E, d):
    """Of the standalone direct gate: threads of a task, and in how many runs the partial sums of a logit are added up."""
    threads, n = (512 if E * d > 1 << 17 else 256), direct_tokens(T) * E
    return threads, 1 if threads // (E // 8) < 64 or 2 * n > threads else min(16, 1 << (threads // n).bit_length() - 1)


def direct_parts(T, E, d):
    """Parts, by experts, of a task of the direct gate inside the layer."""
    if T > 128 or E * d < 1 << 18:
        return 1
    return max(1, min(CUS // T, E // 16, 8))


def part_pieces(E, parts):
    """Pieces of 8 experts in each part."""
    return [E // 8 * (s + 1) // parts - E // 8 * s // parts for s in range(parts)]


def is_exact_alone(T, E, d):
    """moe_route: exact logits of all experts on the fp64 matrix units."""
    if E <= 16:
        return d <= (2048 if T > 2048 and E % 8 == 0 else 1024)
    most = 640 if E <= 32 else 384 if E <= 48 else 192 if E <= 64 else 128
    return d <= (most if T > 2048 else most * 3 // 4 if T > 1024 else most // 2)


def screen_variant(E, d):
    return (1 if d % 128 == 0 else 6) if E <= 32 else 2 if E <= 64 else 3 if E <= 128 else 4 if E <= 192 else 5


def screen_tokens(T):
    return 16 if T > 2048 else 8 if T > 1024 else 4


def form(T, E, d, alone):
    """'direct', 'exact' or ('screen', code variant, tokens per task)."""
    if is_direct(T, E, d, alone):
        return "direct"
    if alone and is_exact_alone(T, E, d):
        return "exact"
    return ("screen", screen_variant(E, d), screen_tokens(T))

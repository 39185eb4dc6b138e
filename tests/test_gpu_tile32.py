"""The tile bodies (32 rows per wave, head_dim 256: 16): their first, last and middle tiles are different code, the reference of the
softmax moves in each of them, and dead slots of the last tile are zeroed in LDS.  Against the fp64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2402_01869_amd import workloads as W
from gpu_common import AttnRunner, make_pool

pytestmark = pytest.mark.gpu

# keys before the chunk: 1 to 3 tiles, and around the pairs of steps that the middle code takes
PREFIXES = (0, 1, 31, 63, 64, 65, 127, 128, 190, 192, 255, 256, 257, 320, 383, 449, 513, 640, 705)


@pytest.mark.parametrize("H,Hkv,D,rows", [(2, 2, 64, 2), (2, 2, 128, 67), (16, 2, 64, 33), (8, 1, 128, 40), (9, 9, 128, 5), (1, 1, 64, 300),
                                           (2, 2, 256, 2), (3, 3, 256, 67), (8, 1, 256, 40), (1, 1, 256, 150)])
@pytest.mark.parametrize("jumps", [(), (40, 97, 129, 200, 290, 350, 410, 480, 600)])
def test_tiles_of_every_number_and_moving_references(H, Hkv, D, rows, jumps):
    """jumps: from each of these keys on the scores grow by some 12 in log2 units, more than the slack of 8, so that the
    accumulated results are rescaled there, in whichever code has the tile."""
    rng = np.random.default_rng(D + rows + len(jumps))
    ctx = [p + rows for p in PREFIXES]
    batch = W.assemble_batch(H, D, 16, sum(-(-c // 16) for c in ctx) + 9, ctx, [rows] * len(ctx), rng, num_kv_heads=Hkv)
    pool_bits, q_bits = W.make_host_inputs(batch, 3 + D, poison_unused=True)
    if jumps:   # dim 0 of every query is 1, of a key its offset
        q_bits[..., 0] = W.f32_to_bf16_bits(np.float32(1.0))
        for s, c in enumerate(ctx):
            for t in range(c):
                level = 8.0 * np.sqrt(D) * sum(t >= j for j in jumps)     # 8 x log2(e) = 11.5 a jump
                pool_bits[batch.block_tables[s, t // 16], 0, :, t % 16, 0] = W.f32_to_bf16_bits(np.float32(level))
    want = oracle.attn_batch(batch, pool_bits, q_bits)
    pool, keep = make_pool(pool_bits, H)
    for part in (1 << 20, 256, 64):
        pool.set_tuning(span_part_tokens=part)
        got = W.bf16_bits_to_f64(AttnRunner(pool, batch, q_bits).run())
        assert np.isfinite(got).all()
        # The path's flat bar, and from a magnitude of 4 on half a unit of the bf16 grid and 2e-3.  A row that has just passed a jump
        # rests on a few keys: its weights, rounded by up to 2^-9, are normalised as rounded, so the result is off by at most
        # 2^-9 of the largest distance between two values, and half a unit of the grid.
        half = np.ldexp(1.0, np.floor(np.log2(np.maximum(np.abs(want), 2.0 ** -30))).astype(np.int64) - 8)
        err, few = np.abs(got - want), 2.0 ** -9 * 2 * 5.0 + half     # N(0, 1) values: below 5
        assert (err <= (few if jumps else np.where(np.abs(want) < 4.0, 1e-2, half + 2e-3))).all(), (part, float(err.max()))
    pool.close()


NONE, NAN, INF, BIG = None, 0x7FC0, 0x7F80, 0x7F7E     # bf16 patterns; BIG: 3.4e38, whose scores overflow


@pytest.mark.parametrize("H,Hkv,D", [(2, 2, 64), (4, 2, 64), (16, 2, 64), (2, 2, 128), (8, 1, 128), (9, 3, 128), (2, 2, 256), (8, 1, 256)])
@pytest.mark.parametrize("jumps", [(), (97, 200, 290, 350, 480, 600, 710)])
def test_non_finite_scores_stay_in_the_rows_that_have_them(H, Hkv, D, jumps):
    """A NaN or an infinity in a query row shows in that row and head alone, one in a key of the chunk only in the rows that see
    the key: the same results are non-finite as on the vector kernel, row by row, and all others are right.  Prefixes put the
    chunk into the first, the last and middle tiles, on one item or on several; jumps: as above."""
    rng = np.random.default_rng(H + D)
    rows, prefixes = 75, (64, 65, 130, 200, 321, 449, 640, 705, 900)
    # row and bits of a query element, or key of the chunk and bits
    bad_q = (NONE, (5, NAN), (20, INF), NONE, (40, NAN), NONE, (70, BIG), NONE, NONE)
    bad_k = ((17, NAN), NONE, NONE, (50, INF), NONE, (2, NAN), NONE, (66, INF), (31, NAN))
    ctx = [p + rows for p in prefixes]
    batch = W.assemble_batch(H, D, 16, sum(-(-c // 16) for c in ctx) + 9, ctx, [rows] * len(ctx), rng, num_kv_heads=Hkv)
    pool_bits, q_bits = W.make_host_inputs(batch, 3 + D, poison_unused=True)
    if jumps:
        q_bits[..., 0] = W.f32_to_bf16_bits(np.float32(1.0))
        for s, c in enumerate(ctx):
            for t in range(c):
                level = 8.0 * np.sqrt(D) * sum(t >= j for j in jumps)
                pool_bits[batch.block_tables[s, t // 16], 0, :, t % 16, 0] = W.f32_to_bf16_bits(np.float32(level))
    for s, (pre, q, k) in enumerate(zip(prefixes, bad_q, bad_k)):
        if q:
            q_bits[s * rows + q[0], (s + 1) % H, 7 * s] = q[1]
        if k:
            pos = pre + k[0]
            pool_bits[batch.block_tables[s, pos // 16], 0, s % Hkv, pos % 16, 5 * s] = k[1]
    pool, keep = make_pool(pool_bits, H)
    run = lambda **tuning: (pool.set_tuning(**tuning), W.bf16_bits_to_f64(AttnRunner(pool, batch, q_bits).run()))[1]
    by_row = run(span_kernel=1)
    fine = np.isfinite(by_row)
    lost = ~fine.all(axis=-1)                              # [row][head]
    assert (lost == ~fine.any(axis=-1)).all()
    for s, (q, k) in enumerate(zip(bad_q, bad_k)):         # as the values were placed
        mine = lost[s * rows:(s + 1) * rows]
        if q:
            assert mine.sum() == 1 and mine[q[0], (s + 1) % H]
        elif k[1] == NAN:
            heads = np.arange(H) // (H // Hkv) == s % Hkv
            assert (mine == (np.arange(rows)[:, None] >= k[0]) & heads).all()
        else:
            assert not mine[:k[0]].any() and mine.any()
    for part in (0, 256, 64):
        got = run(span_part_tokens=part)
        assert np.array_equal(np.isfinite(got), fine), (part, np.argwhere((np.isfinite(got) != fine).any(axis=-1))[:8].tolist())
        # the bars of the test above, and half a unit of the bf16 grid for the vector kernel's rounding
        err, size = np.abs(got - by_row)[fine], np.abs(by_row)[fine]
        assert (err <= (2.0 ** -9 * 2 * 5.0 + size * 2.0 ** -7 if jumps else 1e-2 + size * 2.0 ** -8)).all(), (part, float(err.max()))
    pool.close()

"""Rows of a chunk that see fewer than 64 keys run as units of the tile kernels (one per sequence and pair of query
heads), their weights split into three bf16 parts: compared with the vector kernel (fp32 weights) and the fp64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2402_01869_amd import binding as B
from paper_2402_01869_amd import workloads as W
from gpu_common import AttnRunner, make_pool

pytestmark = pytest.mark.gpu

# (context, chunk): fresh chunks around the 16-row waves and the 64-key limit, and short prefixes before the chunk
EDGES = [(2, 2), (15, 15), (16, 16), (17, 17), (33, 33), (62, 62), (63, 63), (64, 64), (65, 65), (100, 99), (63, 2), (64, 3),
         (48, 17), (80, 40), (300, 300), (64, 2), (40, 1), (500, 1)]


def _run(batch, pool_bits, q_bits, **tuning):
    pool, keep = make_pool(pool_bits, batch.num_heads)
    pool.set_tuning(**tuning)
    if tuning.get("span_kernel") != 1:
        how = pool.plan_launches(B.HostDesc.from_batch(batch))
        assert how["n_few_items"] > 0 and how["side_by_side"] == ("row_launch" in tuning)
    out = W.bf16_bits_to_f64(AttnRunner(pool, batch, q_bits).run())
    pool.close()
    return out


@pytest.mark.parametrize("H,Hkv,D", [(1, 1, 64), (5, 5, 64), (3, 3, 128), (10, 10, 128), (16, 2, 128), (6, 2, 128), (2, 2, 256), (3, 1, 256)])
def test_few_key_rows_match_the_vector_kernel(H, Hkv, D):
    rng = np.random.default_rng(H + 7 * Hkv + D)
    ctx, q_len = [c for c, _ in EDGES], [n for _, n in EDGES]
    batch = W.assemble_batch(H, D, 16, 200, ctx, q_len, rng, num_kv_heads=Hkv)
    pool_bits, q_bits = W.make_host_inputs(batch, 5 + D, poison_unused=True)
    want = oracle.attn_batch(batch, pool_bits, q_bits)
    rows = np.concatenate([np.arange(c - n, c) for c, n in EDGES]) < 63   # rows that see fewer than 64 keys
    by_row = _run(batch, pool_bits, q_bits, span_kernel=1)
    # alone, beside the slim row or group kernel, and with another limit
    for tuning in (dict(), dict(row_launch=2), dict(row_launch=3, row_slots=9), dict(mfma_min_keys=30)):
        got = _run(batch, pool_bits, q_bits, **tuning)
        assert np.isfinite(got).all()
        mine = rows if tuning.get("mfma_min_keys", 64) == 64 else np.concatenate([np.arange(c - n, c) for c, n in EDGES]) < 29
        # two results that agree to 2^-16 relative round to neighbouring bf16 values at most
        assert (np.abs(got - by_row)[mine] <= np.abs(by_row)[mine] * 2.0 ** -7 + 1e-5).all(), tuning
        # and each is within half a unit of the bf16 grid of the oracle, up to the fp32 sums
        assert (np.abs(got - want)[mine] <= np.abs(want)[mine] * 2.0 ** -8 * 1.001 + 1e-4).all(), tuning
        # An error of e before the rounding to bf16 (spacing 2^-8 to 2^-7) changes some e / 2^-8 of the values: fp32 sums of up
        # to 63 terms 0.01 %, weights of 16 bits (2^-18 in the mean) 0.1 to 0.2 %.
        nearest = W.bf16_bits_to_f64(W.f32_to_bf16_bits(want.astype(np.float32)))
        assert (got != nearest)[mine].mean() <= 5e-4, (tuning, (got != nearest)[mine].mean(), (by_row != nearest)[mine].mean())


@pytest.mark.parametrize("D", [64, 128, 256])
def test_few_key_rows_with_infinite_and_nan_values(D):
    """An infinite or NaN value shows in exactly the rows that see its key, as on the vector kernel."""
    H, few = 3, 50 + 63 + 20 + 63      # the last chunk's other rows are a tile item, beside which the units run
    batch = W.assemble_batch(H, D, 16, 64, [50, 63, 30, 90], [50, 63, 20, 90], np.random.default_rng(D))
    pool_bits, q_bits = W.make_host_inputs(batch, 9, poison_unused=True)
    for s, key, head, dim, bits in ((0, 20, 0, 3, 0x7F80), (0, 33, 1, D - 1, 0xFF80), (1, 62, 2, 17, 0x7FC0), (2, 12, 0, 0, 0x7F80)):
        pool_bits[batch.block_tables[s, key // 16], 1, head, key % 16, dim] = bits
    by_row = _run(batch, pool_bits, q_bits, span_kernel=1)[:few]
    got = _run(batch, pool_bits, q_bits)[:few]
    fine = np.isfinite(by_row)
    assert not fine.all() and fine.any()
    assert np.array_equal(np.isnan(got), np.isnan(by_row)) and np.array_equal(got[~fine & ~np.isnan(got)], by_row[~fine & ~np.isnan(by_row)])
    got, by_row = got[fine], by_row[fine]
    assert (np.abs(got - by_row) <= np.abs(by_row) * 2.0 ** -7 + 1e-5).all()

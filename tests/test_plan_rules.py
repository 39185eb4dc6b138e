"""Rules of the launch planner that depend on how much of the chip a batch fills (host only)."""
import numpy as np
import pytest

from paper_2402_01869_amd import binding as B
from paper_2402_01869_amd import workloads as W


def _plan(H, Hkv, D, ctx, q_len, **tuning):
    rng = np.random.default_rng(1)
    blocks = sum(-(-c // 16) for c in ctx) + 4
    batch = W.assemble_batch(H, D, 16, blocks, ctx, q_len, rng, num_kv_heads=Hkv)
    pool = B.KvPool(B.make_cfg(blocks, H, D, num_kv_heads=Hkv), 0x10000, blocks * 64 * Hkv * D)   # base never dereferenced
    pool.set_tuning(**tuning)
    desc = B.HostDesc.from_batch(batch)
    plan = pool.plan_image(desc)
    plan["workspace"] = pool.workspace_bytes(desc)
    pool.close()
    return plan


@pytest.mark.parametrize("H,Hkv,D,ctx,split", [
    (40, 40, 128, [3000], True),            # 40 workgroups on 256 CUs: several partitions per row
    (64, 8, 128, [1000, 4500, 8000], True),
    (16, 16, 256, [4096] * 4, True),
    (40, 40, 128, [200] * 3, False),        # short rows: the merge would cost more than it gives
    (4, 4, 64, [128, 100], False),
    (40, 40, 128, [4000] * 26, False),      # four rounds of whole rows
    (64, 8, 128, [4000] * 256, False),
])
def test_decode_rows_are_split_only_when_they_leave_the_chip_idle(H, Hkv, D, ctx, split):
    plan = _plan(H, Hkv, D, ctx, [1] * len(ctx))
    part = plan["row_part_tokens"]
    assert part % 64 == 0 and 128 <= part <= 4096
    assert (part < max(ctx)) == split or max(ctx) > 4096
    assert plan["n_row_items"] == sum(-(-c // part) for c in ctx)
    forced = _plan(H, Hkv, D, ctx, [1] * len(ctx), decode_part_tokens=1024)   # the caller's choice stands
    assert forced["row_part_tokens"] == 1024

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
    assert (part < min(max(ctx), 4096)) == split          # 4096 keys: the most an item can hold
    assert plan["n_row_items"] == sum(-(-c // part) for c in ctx)
    forced = _plan(H, Hkv, D, ctx, [1] * len(ctx), decode_part_tokens=1024)   # the caller's choice stands
    assert forced["row_part_tokens"] == 1024


@pytest.mark.parametrize("H,Hkv,D,ctx,q_len,split", [
    (64, 8, 128, [3012], [512], True),                     # 128 workgroups of 48 steps on 256 CUs
    (16, 2, 64, [8900] * 3, [67] * 3, True),
    (4, 4, 256, [6000], [100], True),
    (40, 40, 128, [512], [512], False),                    # a fresh chunk: the merge would cost more than it gives
    (4, 4, 64, [128, 96], [32, 32], False),
    (64, 8, 128, [3012] * 8, [512] * 8, False),            # four rounds of whole tiles
    (40, 40, 128, [4000] * 100 + [3012], [1] * 100 + [512], False),   # the decode rows take longer anyway
])
def test_spans_are_split_only_when_their_tiles_leave_the_chip_idle(H, Hkv, D, ctx, q_len, split):
    plan = _plan(H, Hkv, D, ctx, q_len)
    part, longest = plan["span_part_tokens"], max(c for c, n in zip(ctx, q_len) if n > 1)
    assert part % 64 == 0 and part >= 256
    assert (part < longest) == split
    assert (plan["partial_slots"] > 0) == split
    whole = _plan(H, Hkv, D, ctx, q_len, span_part_tokens=1 << 20)      # the caller's choice stands
    assert whole["span_part_tokens"] == 1 << 20 and whole["partial_slots"] == 0


def test_few_key_rows_become_units_only_beside_tiles_or_in_numbers():
    """Their row items stay in the plan either way; the units are a section of the image."""
    tiny = _plan(16, 16, 256, [2, 2, 2, 20], [2, 2, 2, 1])      # 6 rows x 16 heads: the vector kernel's launch takes them
    many = _plan(16, 16, 256, [60] * 4, [60] * 4)
    beside = _plan(16, 16, 256, [2, 300], [2, 300])
    for plan, rows in ((tiny, 7), (many, 240), (beside, 65)):
        assert plan["n_row_items"] == rows == plan["n_vector_row_items"]
    assert tiny["off_merge_items"] - tiny["off_tile_items"] < 256       # no tile items, no units
    assert many["off_merge_items"] > many["off_tile_items"]             # units only
    assert beside["off_merge_items"] - beside["off_tile_items"] >= 512  # both


@pytest.mark.parametrize("H,Hkv,D,n,keys,n_span,pair", [
    # decode rows x keys beside chunks of 512 rows on 1500 keys; measured side by side / one after the other, us
    (40, 40, 128, 43, 560, 2, True),      # 112 / 145
    (40, 40, 128, 46, 350, 4, True),      # 140 / 179
    (16, 16, 256, 100, 200, 3, True),     # 108 / 140
    (32, 32, 64, 54, 1100, 6, True),      # 132 / 170
    (64, 8, 128, 40, 1500, 2, True),      # 98 / 119
    (16, 4, 128, 54, 1500, 5, True),      # 78 / 101
    (40, 40, 128, 604, 40, 2, False),     # 318 / 161: the queue, not the memory
    (32, 32, 64, 1007, 40, 6, False),     # 413 / 155
    (40, 40, 128, 483, 100, 2, False),    # 299 / 239
    (16, 16, 256, 755, 40, 2, False),     # 204 / 165
])
def test_batches_run_side_by_side_where_that_is_faster(H, Hkv, D, n, keys, n_span, pair):
    ctx, q_len = [keys] * n + [2012] * n_span, [1] * n + [512] * n_span
    assert bool(_plan(H, Hkv, D, ctx, q_len)["side_by_side"]) == pair
    # one request that has just begun to decode changes nothing for the others
    assert bool(_plan(H, Hkv, D, [40] + ctx, [1] + q_len)["side_by_side"]) == pair


@pytest.mark.parametrize("H,Hkv,D,n,keys,n_span,span,prefix,pair", [
    # one kind of work is most of the call; measured side by side / one after the other, us
    (64, 8, 128, 196, 15062, 12, 71, 2, False),      # 1878 / 1808 a layer
    (32, 32, 64, 224, 3000, 1, 256, 500, False),     # 1051 / 800
    (32, 32, 64, 56, 12000, 2, 400, 500, False),     # 1023 / 794
    (16, 16, 256, 1, 100, 8, 2048, 2048, True),      # 1087 / 1171
    (16, 16, 256, 1, 100, 8, 2048, 4096, True),      # 1782 / 1890
    (16, 16, 256, 1, 100, 4, 1024, 2048, False),     # 229 / 220
])
def test_batches_of_mostly_one_kind(H, Hkv, D, n, keys, n_span, span, prefix, pair):
    assert bool(_plan(H, Hkv, D, [keys] * n + [prefix + span] * n_span, [1] * n + [span] * n_span)["side_by_side"]) == pair


@pytest.mark.parametrize("H,Hkv,D,n,keys,n_span,prefix,split", [
    # measured side by side with whole rows / in items of 1024 keys, us
    (40, 40, 128, 4, 4000, 4, 2500, False),      # the tiles lead
    (40, 40, 128, 5, 4000, 4, 2500, False),      # 200 / 204
    (40, 40, 128, 8, 4000, 4, 2500, False),
    (64, 8, 128, 63, 1500, 4, 1500, False),      # 157 / 164 (768 keys)
    (40, 40, 128, 3, 4000, 2, 2000, True),       # 116 / 94: 120 long items beside 160 tiles on 256 CUs
    (40, 40, 128, 7, 4000, 3, 1500, True),       # 159 / 132: the second round of long items has 24
    (16, 16, 256, 6, 4000, 2, 1500, True),       # 161 / 113
])
def test_rows_beside_tiles_are_split_where_that_ends_sooner(H, Hkv, D, n, keys, n_span, prefix, split):
    plan = _plan(H, Hkv, D, [keys] * n + [prefix + 512] * n_span, [1] * n + [512] * n_span)
    assert plan["side_by_side"] and (plan["row_part_tokens"] < 4096) == split
    assert (plan["row_items"][:, 4] >= 0).any() == split


@pytest.mark.parametrize("H,Hkv,D,n,keys,n_span,span,prefix,pair,split", [
    # plans that follow from the rates of the tile kernels as they are; measured this way / as planned with the rates of the
    # kernels before them, us
    (16, 16, 256, 1, 8000, 3, 90, 3000, False, True),    # 70.5 / 81.2 side by side
    (16, 16, 256, 86, 350, 2, 512, 1500, True, False),   # 113 / 125 with the chunks split
    (64, 8, 128, 72, 1500, 1, 512, 1500, True, False),   # 109 / 129 with the chunks split
])
def test_plans_follow_the_rates_of_the_tile_kernels(H, Hkv, D, n, keys, n_span, span, prefix, pair, split):
    plan = _plan(H, Hkv, D, [keys] * n + [prefix + span] * n_span, [1] * n + [span] * n_span)
    assert bool(plan["side_by_side"]) == pair
    assert (plan["span_part_tokens"] < prefix + span) == split


@pytest.mark.parametrize("H,Hkv,ctx,q_len,kernel", [
    (40, 40, [3000, 16384], [1, 2048], 1),     # 2048 span rows row by row
    (64, 8, [3000, 700], [1, 100], 1),
    (64, 8, [3000, 6000], [1, 1], 2),          # decode rows as one-row tiles
    (64, 8, [3000, 16384], [1, 512], 2),
    (64, 8, [3000, 40, 6000, 2000, 2000], [1, 1, 1, 512, 512], 2),   # ... beside one that is a row item
])
def test_the_partition_of_a_few_decode_rows_is_not_put_on_other_rows(H, Hkv, ctx, q_len, kernel):
    plan, whole = (_plan(H, Hkv, 128, ctx, q_len, span_kernel=kernel, **t) for t in (dict(), dict(decode_part_tokens=4096)))
    assert plan["row_part_tokens"] == 4096 and plan["workspace"] == whole["workspace"]


@pytest.mark.parametrize("n_span", [1, 2, 3])
def test_one_short_decode_row_leaves_a_grouped_batch_side_by_side(n_span):
    ctx = [2000] * 64 + [2500] * n_span
    for short in (0, 1, 5):
        plan = _plan(64, 8, 128, [40] * short + ctx[short:], [1] * 64 + [512] * n_span)
        assert plan["side_by_side"] and plan["group_launch"] == B.IC_LAUNCH_SLIM


@pytest.mark.parametrize("H,Hkv,D,ctx,q_len", [(4, 4, 64, [16, 100, 64, 90], [1, 1, 32, 32]), (16, 16, 256, [200, 700], [200, 1]),
                                               (64, 8, 128, [700, 300], [1, 40]), (6, 2, 128, [9, 200], [1, 100])])
def test_asking_for_persistent_rows_asks_for_both_kernels_side_by_side(H, Hkv, D, ctx, q_len):
    """By itself a small batch runs one kernel after the other; with persistent row workgroups asked for it runs the pair."""
    assert not _plan(H, Hkv, D, ctx, q_len)["side_by_side"] and not _plan(H, Hkv, D, ctx, q_len, row_launch=1)["side_by_side"]
    for tuning in (dict(row_launch=2), dict(row_launch=3), dict(row_slots=7)):
        plan = _plan(H, Hkv, D, ctx, q_len, **tuning)
        assert plan["side_by_side"] and plan["tile_launch"] == B.IC_LAUNCH_PERSISTENT
        assert {plan["row_launch"], plan["group_launch"]} <= {B.IC_LAUNCH_NONE, B.IC_LAUNCH_SLIM}
        assert plan["n_merged_inside"] == 0                  # from a queue the merge kernel merges
        assert not _plan(H, Hkv, D, ctx, q_len, serial_spans=1, **tuning)["side_by_side"]
        assert not _plan(H, Hkv, D, ctx[:1], q_len[:1], **tuning)["side_by_side"]     # nothing to run beside


@pytest.mark.parametrize("H,Hkv,D", [(4, 4, 64), (5, 5, 128), (2, 2, 256), (64, 8, 128), (6, 2, 64)])
def test_few_items_and_split_slots_of_the_image(H, Hkv, D):
    """Every few item covers consecutive rows of one sequence, each such row exactly once; every partial slot of a row that
    its last partition merges names that row's merge item; the arrival counters start at zero."""
    rng = np.random.default_rng(H + Hkv + D)
    seen_units = seen_split = 0
    for trial in range(40):
        n = int(rng.integers(1, 7))
        ctx = [int(rng.integers(1, 70)) if rng.random() < 0.4 else int(rng.integers(64, 5000)) for _ in range(n)]
        q_len = [1 if rng.random() < (0.5, 1.0)[trial % 2] else int(rng.integers(1, min(c, 400) + 1)) for c in ctx]
        plan = _plan(H, Hkv, D, ctx, q_len)
        rows, few = plan["row_items"], plan["few_items"]
        first = plan["n_vector_row_items"] - plan["n_few_rows"]
        assert few[:, 1].sum() == plan["n_few_rows"]
        for at, k in few.tolist():
            assert at == first and 1 <= k <= 63            # back to back, behind the vector kernel's items
            first += k
            seq, pos = rows[at, 0], rows[at:at + k, 3]
            assert (rows[at:at + k, 0] == seq).all() and q_len[seq] > 1
            assert (rows[at:at + k, 1] == rows[at, 1] + np.arange(k)).all() and (pos == pos[0] + np.arange(k)).all()
            assert pos[0] == ctx[seq] - q_len[seq] + 1 and pos[-1] <= 63
            assert (rows[at:at + k, 2] == 0).all() and (rows[at:at + k, 4] == -1).all()
        assert first == plan["n_vector_row_items"]
        assert bool(len(few)) <= bool(plan["tile_launch"])
        inside = plan["n_merged_inside"]
        for mi, (qrow, slot0, nparts, _) in enumerate(plan["merge_items"].tolist()[:inside]):
            assert (plan["slot_merge"][slot0:slot0 + nparts] == mi).all()
            mine = rows[rows[:, 1] == qrow]
            assert sorted(mine[:, 4].tolist()) == list(range(slot0, slot0 + nparts))
        assert plan["n_split_slots"] == sum(m[2] for m in plan["merge_items"].tolist()[:inside])
        assert len(plan["arrived"]) == inside * plan["n_split_units"] and not plan["arrived"].any()
        seen_units += len(few)
        seen_split += inside
    assert seen_units and seen_split


def test_whole_rows_of_the_group_kernel_do_not_pay_for_the_merging_end():
    """The build that runs rows which are not split spills no more than the kernel alone does (its key loop included); the end
    that merges is in a build of its own."""
    import os
    import re
    import shutil
    import subprocess
    import tempfile
    if not shutil.which("hipcc"):
        pytest.skip("hipcc not on PATH")
    src = os.path.join(os.path.dirname(os.path.abspath(B.__file__)), "csrc", "attn_group.hip")
    with tempfile.TemporaryDirectory() as tmp:
        r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                            "-packed-fp32-ops", "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o", os.path.join(tmp, "g.o")],
                           capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    scratch, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: \S*group_attn_kernelI(\S+?)EEEv", line)
        name = m.group(1) if m else None if "Function Name" in line else name
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and name:
            scratch[name] = int(m.group(1))
    assert scratch["Li64ELb0"] == scratch["Li128ELb0"] == 0 and scratch["Li256ELb0"] <= 124, scratch


def test_the_benchmark_names_the_kernels_that_run():
    """The report's kernel names follow the planner's launches, not the tuning alone."""
    import types
    import bench
    for H, Hkv, D, ctx, q_len, want in [
            (4, 4, 64, [16, 100, 64, 90], [1, 1, 32, 32], ("row_attn_kernel<64>", "tile_persist_kernel<64, false>", False)),
            (40, 40, 128, [3000], [1], ("row_attn_kernel<128>", None, False)),               # split, merged by its last partition
            (40, 40, 128, [4000] * 40, [1] * 40, ("row_persist_kernel<128>", None, False)),
            (16, 16, 256, [600, 900], [300, 1], ("row_attn_kernel<256>", "tile_attn_kernel<256>", False)),
            (40, 40, 128, [3000] * 60 + [3000] * 8, [1] * 60 + [512] * 8, ("row_persist_slim_kernel<128>", "tile_persist_kernel<128, true>", True))]:
        rng = np.random.default_rng(1)
        blocks = sum(-(-c // 16) for c in ctx) + 4
        batch = W.assemble_batch(H, D, 16, blocks, ctx, q_len, rng, num_kv_heads=Hkv)
        pool = B.KvPool(B.make_cfg(blocks, H, D, num_kv_heads=Hkv), 0x10000, blocks * 64 * Hkv * D)
        names = bench.attention_kernel_names(pool, B.HostDesc.from_batch(batch), types.SimpleNamespace(head_dim=D, num_heads=H, kv_heads=Hkv))
        assert names["row"] == want[0] and names["side_by_side"] == want[2]
        assert want[1] is None or names["tile"] == want[1]
        pool.close()


@pytest.mark.parametrize("H,Hkv,D,ctx", [(5, 5, 64, [700, 3000, 90, 1500]), (3, 3, 128, [4096, 130, 2000]), (2, 2, 256, [1000, 2600]),
                                         (16, 2, 128, [5000, 300, 64]), (6, 2, 64, [2500, 40]), (32, 1, 256, [1800, 700])])
@pytest.mark.gpu
def test_rows_merged_by_their_last_partition(H, Hkv, D, ctx):
    """The split the planner chooses for a few decode rows (merged inside the row or group kernel) against the oracle, and
    the merge kernel's result for the same partitions; several layers and repetitions from one plan, whose arrival
    counters have to come back to zero."""
    import torch
    import oracle
    from gpu_common import AttnRunner, make_pool, max_abs_err, from_dev_bits
    batch = W.assemble_batch(H, D, 16, 800, ctx, [1] * len(ctx), np.random.default_rng(D), num_kv_heads=Hkv)
    pool_bits, q_bits = W.make_host_inputs(batch, 3 + H, poison_unused=True)
    want = oracle.attn_batch(batch, pool_bits, q_bits)
    pool, keep = make_pool(pool_bits, H)
    desc = B.HostDesc.from_batch(batch)
    part = pool.plan_image(desc)["row_part_tokens"]
    assert part < max(ctx)                                        # the plan does split
    r = AttnRunner(pool, batch, q_bits)
    once = r.run().copy()
    assert max_abs_err(once, want) <= 1e-2
    ws = torch.empty(pool.workspace_bytes(desc), dtype=torch.uint8, device="cuda:0")
    plan = pool.plan_create(desc, ws.data_ptr(), ws.numel())
    for _ in range(20):
        r.out.fill_(0x7FFF)
        for _ in range(3):
            pool.paged_attn_planned(plan, r.q.data_ptr(), r.out.data_ptr())
        torch.cuda.synchronize()
        assert np.array_equal(from_dev_bits(r.out), once)
    plan.close()
    pool.set_tuning(decode_part_tokens=part)                      # the same partitions, merged by the merge kernel
    assert np.array_equal(AttnRunner(pool, batch, q_bits).run(), once)
    pool.close()


@pytest.mark.parametrize("H,Hkv,D,ctx,q_len", [(5, 5, 128, [3000, 90], [1, 1]), (16, 2, 128, [5000, 700], [1, 100]),
                                               (4, 4, 64, [2600, 300], [40, 300])])
@pytest.mark.gpu
def test_a_workspace_without_room_for_the_split_runs_whole_rows(H, Hkv, D, ctx, q_len):
    """A workspace large enough for whole rows and tiles (allocated for another batch, say) is accepted, and few-key rows stay
    units of the tile kernel as long as their few bytes fit too."""
    import torch
    import oracle
    from gpu_common import from_dev_bits, make_pool, max_abs_err, to_dev_bits
    batch = W.assemble_batch(H, D, 16, 512, ctx, q_len, np.random.default_rng(D), num_kv_heads=Hkv)
    pool_bits, q_bits = W.make_host_inputs(batch, 21, poison_unused=True)
    want = oracle.attn_batch(batch, pool_bits, q_bits)
    pool, keep = make_pool(pool_bits, H)
    desc = B.HostDesc.from_batch(batch)
    full = pool.workspace_bytes(desc)
    pool.set_tuning(decode_part_tokens=4096, span_part_tokens=1 << 20)
    whole = pool.workspace_bytes(desc)
    if max(ctx) <= 4096:
        assert pool.plan_query(desc)["partial_slots"] == 0
    few = pool.plan_launches(desc)["n_few_items"]
    pool.set_tuning()
    assert whole < full and few == (1 if q_len == [40, 300] else 0)
    q, ws = to_dev_bits(q_bits), torch.empty(full, dtype=torch.uint8, device="cuda:0")
    for planned, room in ((False, whole), (True, whole), (False, whole - 256 * few), (True, whole - 256 * few)):
        pool.prof_begin(16)
        out = torch.full(tuple(q_bits.shape), 0x7FFF, dtype=torch.int16, device="cuda:0")
        if planned:
            plan = pool.plan_create(desc, ws.data_ptr(), room)
            pool.paged_attn_planned(plan, q.data_ptr(), out.data_ptr())
        else:
            pool.paged_attn_mixed(desc, q.data_ptr(), out.data_ptr(), ws.data_ptr(), room)
        torch.cuda.synchronize()
        assert max_abs_err(from_dev_bits(out), want) <= 1e-2
        if few:      # no decode rows here: the row kernel runs for few-key rows that are not units
            assert pool.prof_end()["row"]["launches"] == (0 if room == whole else 1)
    plan.close()
    assert pool.paged_attn_mixed(desc, q.data_ptr(), out.data_ptr(), ws.data_ptr(), 1024, check=False) == B.IC_ESIZE
    pool.close()

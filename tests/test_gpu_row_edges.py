"""Edges of the row-splitting kernels: rows of a wave that is not full (16-byte pieces that lanes exchange, sixteen rows at
once), block ids of segments longer than the kernel holds at once, the orders and queues of whole sequences' row groups, the
merge in the launch and behind it (and decoding steps, which have none behind), against the oracle."""
import numpy as np
import pytest
import torch

import aspd_workloads as W
from oracle import attend
from oracle.sequence_layout import replay_layout

pytestmark = pytest.mark.gpu

TOL, LSE_TOL = 2e-2, 2e-3    # bf16 weights and results, 2^-9 each


@pytest.mark.parametrize("heads", [(8, 8, 128), (4, 4, 64), (6, 2, 128)])
@pytest.mark.parametrize("tokens", [1, 15, 16, 17, 31, 32, 33, 79, 271])
def test_last_wave_of_a_row_group(heads, tokens):
    from gpu_drive import GpuBatch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_08895_amd import binding as A
    layouts = [[(0, tokens)], [(0, tokens // 2 + 1)]]
    wl = W.random_small(seed=5900 + tokens, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2], batch=2,
                        prefix_range=(tokens, tokens), branches_range=(1, 1), branch_len_range=(1, 1))
    tt, meta = replay_layout(wl.block_tables, wl.block_size, layouts)
    gb = GpuBatch(wl)
    step = A.aspd_build_sequence_meta(gb.kv, gb.state, gb._dev_i32([0, 1, 2]), gb._dev_i32([0, 0]),
                                      gb._dev_i32([r[0][1] for r in layouts]), NQ=meta.NQ)
    q = wl.draw_q(meta.NQ)
    # a row more than there are, which nothing may write
    out = torch.full((meta.NQ + 1, *q.shape[1:]), float("nan"), dtype=q.dtype, device=gb.dev)
    lse = torch.full((meta.NQ + 1, heads[0]), float("nan"), dtype=torch.float32, device=gb.dev)
    A.aspd_attn_full_sequence(gb.kv, gb.state, step, q.to(gb.dev), gb.workspace, out=out, lse=lse)
    assert torch.isnan(out[meta.NQ]).all() and torch.isnan(lse[meta.NQ]).all()
    ref, ref_lse = attend(tt, meta, q, wl.k_cache, wl.v_cache)
    assert np.abs(out[:meta.NQ].float().cpu().numpy() - ref).max() <= TOL
    assert np.abs(lse[:meta.NQ].cpu().numpy() - ref_lse).max() <= LSE_TOL


@pytest.mark.parametrize("heads", [(2, 2, 128), (2, 1, 64)])
@pytest.mark.parametrize("tokens", [4031, 4064, 4097, 4129, 8225])
def test_block_ids_of_long_segments(heads, tokens):
    """The kernel holds the block ids of 64 groups of four pages, the first of group -1, and reads them again from then on:
    key ranges that end before, at and behind those lines, one workgroup each; rows in front of and behind the line."""
    from gpu_drive import GpuBatch
    from paper_2508_08895_amd import binding as A
    wl = W.random_small(seed=6100 + tokens, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2], batch=1,
                        prefix_range=(tokens, tokens), branches_range=(1, 1), branch_len_range=(1, 1))
    tt, meta = replay_layout(wl.block_tables, wl.block_size, [[(0, tokens)]])
    gb = GpuBatch(wl)
    step = A.aspd_build_sequence_meta(gb.kv, gb.state, gb._dev_i32([0, 1]), gb._dev_i32([0]), gb._dev_i32([tokens]),
                                      NQ=meta.NQ, max_workgroups=2)
    q = wl.draw_q(meta.NQ)
    out = A.aspd_attn_full_sequence(gb.kv, gb.state, step, q.to(gb.dev), gb.workspace)
    rows = sorted({0, 31, 4000, *range(4020, min(tokens, 4100), 7), *range(tokens - 40, tokens)})
    ref, _ = attend(tt, meta, q, wl.k_cache, wl.v_cache, rows=rows)
    got = out.float().cpu().numpy()
    assert np.isfinite(got).all()
    assert np.abs(got[rows] - ref[rows]).max() <= TOL


@pytest.mark.parametrize("heads", [(1, 1, 64), (4, 2, 128), (3, 3, 64), (8, 4, 64), (12, 6, 64), (8, 8, 128), (32, 16, 64)])
@pytest.mark.parametrize("cap", [1, 3, 9])
def test_row_groups_from_a_queue_per_xcd(heads, cap):
    """Every row group of every head is computed, whatever the heads' number has in common with the queues', with fewer
    workgroups than queues and with more; the counters are left at zero (the second call finds the same)."""
    from gpu_drive import GpuBatch
    from paper_2508_08895_amd import binding as A
    qpg = 256 // (heads[0] // heads[1])
    need = 12 * cap * qpg // heads[1] + 1          # tokens from which on there is a queue per XCD
    lengths = [need // 2, 0, need // 8 + 1, need // 2 + 37, 5]
    wl = W.random_small(seed=6300 + cap, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2], batch=len(lengths),
                        prefix_range=(max(lengths), max(lengths)), branches_range=(1, 1), branch_len_range=(1, 1))
    layouts = [[(0, n)] for n in lengths]
    tt, meta = replay_layout(wl.block_tables, wl.block_size, layouts)
    gb = GpuBatch(wl)
    step = A.aspd_build_sequence_meta(gb.kv, gb.state, gb._dev_i32(range(len(lengths) + 1)), gb._dev_i32([0] * len(lengths)),
                                      gb._dev_i32(lengths), NQ=meta.NQ, max_workgroups=cap)
    groups = sum(-(-n // qpg) for n in lengths)
    assert groups * heads[1] >= 12 * cap
    q = wl.draw_q(meta.NQ)
    outs = []
    for _ in range(2):
        out = torch.full(q.shape, float("nan"), dtype=q.dtype, device=gb.dev)
        A.aspd_attn_full_sequence(gb.kv, gb.state, step, q.to(gb.dev), gb.workspace, out=out)
        assert int(gb.workspace[:4096].view(torch.int32).abs().sum().item()) == 0
        outs.append(out)
    assert torch.equal(outs[0], outs[1]) and torch.isfinite(outs[0]).all()
    rows = list(range(0, meta.NQ, 1 if meta.NQ < 600 else 17))
    ref, _ = attend(tt, meta, q, wl.k_cache, wl.v_cache, rows=rows)
    assert np.abs(outs[0].float().cpu().numpy()[rows] - ref[rows]).max() <= TOL


@pytest.mark.parametrize("heads", [(32, 8, 128), (8, 2, 64), (4, 4, 128)])
@pytest.mark.parametrize("batch,prefix,branches,chunk", [(1, 900, 3, 11), (1, 1300, 2, 8), (2, 700, 4, 16), (1, 4200, 5, 17),
                                                        (1, 8300, 2, 30), (3, 300, 9, 3)])
@pytest.mark.parametrize("cap", [0, 40])
def test_partial_results_merged_behind_the_launch(heads, batch, prefix, branches, chunk, cap):
    """Chunks of few sequences, whose items have from two parts to 34 (those of up to 48 rows a KV head run the streaming
    kernel): merged by a launch of its own where there are four workgroups an item, with a share of the rows from none to a
    whole round (grids capped too); every row, and the bits of a second call."""
    from gpu_drive import GpuBatch
    from oracle_drive import table_at
    from paper_2508_08895_amd import binding as A
    wl = W.random_small(seed=6500 + prefix, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2], batch=batch,
                        prefix_range=(prefix, prefix + 90), branches_range=(branches, branches), branch_len_range=(1, 9),
                        extra_tokens_per_branch=chunk + 1)
    gb = GpuBatch(wl)
    gb.grow_to(wl.branch_len)
    tt = table_at(wl, wl.branch_len)
    new = np.full(wl.NB, chunk, dtype=np.int32)
    meta = tt.append_parallel(new)
    step = A.aspd_build_branch_meta(gb.kv, gb.state, A.STAGE_PARALLEL, gb._dev_i32(new), NQ=meta.NQ,
                                    max_new_per_seq=branches * chunk, max_workgroups=cap)
    q = wl.draw_q(meta.NQ)
    out = torch.full((meta.NQ + 1, *q.shape[1:]), float("nan"), dtype=q.dtype, device=gb.dev)
    lse = torch.full((meta.NQ + 1, heads[0]), float("nan"), dtype=torch.float32, device=gb.dev)
    A.aspd_attn_branch_chunk(gb.kv, gb.state, step, q.to(gb.dev), gb.workspace, out=out, lse=lse)
    first = out.clone()
    A.aspd_attn_branch_chunk(gb.kv, gb.state, step, q.to(gb.dev), gb.workspace, out=out, lse=lse)
    assert torch.equal(out[:meta.NQ], first[:meta.NQ])
    assert torch.isnan(out[meta.NQ]).all() and torch.isnan(lse[meta.NQ]).all()
    ref, ref_lse = attend(tt, meta, q, wl.k_cache, wl.v_cache)
    assert np.abs(out[:meta.NQ].float().cpu().numpy() - ref).max() <= TOL
    assert np.abs(lse[:meta.NQ].cpu().numpy() - ref_lse).max() <= LSE_TOL


@pytest.mark.parametrize("heads,prefix,branches", [((32, 8, 128), 4300, 9), ((32, 8, 128), 4100, 12), ((24, 4, 128), 9000, 7),
                                                   ((16, 4, 64), 9100, 10), ((16, 4, 64), 6000, 10), ((32, 8, 128), 2000, 12)])
def test_decode_with_three_tiles_and_many_parts(heads, prefix, branches):
    """One token of 33 to 48 rows a KV head behind key ranges of ten to 35 parts."""
    from gpu_drive import GpuBatch
    from oracle_drive import table_at
    from paper_2508_08895_amd import binding as A
    wl = W.random_small(seed=6700 + prefix + branches, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2], batch=1,
                        prefix_range=(prefix, prefix), branches_range=(branches, branches), branch_len_range=(1, 9))
    gb = GpuBatch(wl)
    gb.grow_to(wl.branch_len)
    tt = table_at(wl, wl.branch_len)
    for _ in range(2):
        new = np.ones(wl.NB, dtype=np.int32)
        meta = tt.append_parallel(new)
        step = A.aspd_build_branch_meta(gb.kv, gb.state, A.STAGE_PARALLEL, gb._dev_i32(new), NQ=meta.NQ, max_new_per_seq=branches)
        q = wl.draw_q(meta.NQ)
        out = torch.full((meta.NQ + 1, *q.shape[1:]), float("nan"), dtype=q.dtype, device=gb.dev)
        lse = torch.full((meta.NQ + 1, heads[0]), float("nan"), dtype=torch.float32, device=gb.dev)
        A.aspd_attn_parallel_decode(gb.kv, gb.state, step, q.to(gb.dev), gb.workspace, out=out, lse=lse)
        assert torch.isnan(out[meta.NQ]).all() and torch.isnan(lse[meta.NQ]).all()
        ref, ref_lse = attend(tt, meta, q, wl.k_cache, wl.v_cache)
        assert np.abs(out[:meta.NQ].float().cpu().numpy() - ref).max() <= TOL
        assert np.abs(lse[:meta.NQ].cpu().numpy() - ref_lse).max() <= LSE_TOL


@pytest.mark.parametrize("heads,prefix,branches,hint", [((32, 8, 128), 300, 12, True), ((32, 8, 128), 300, 4, False),
                                                        ((32, 8, 128), 4100, 4, False), ((16, 4, 64), 9100, 10, True),
                                                        ((24, 4, 128), 2000, 7, True)])
@pytest.mark.parametrize("columns", [0, 1024])
@pytest.mark.parametrize("static", [False, True])
def test_decode_is_one_launch(heads, prefix, branches, hint, columns, static):
    """Whatever the width of the block table, with the bound on a step's tokens and without: an attention call of a decoding
    step that brings its plan launches one kernel.  (A second one for the merge, chosen by the table's width, cost steps behind
    short contexts 2 us a layer.)"""
    from gpu_drive import GpuBatch, kernels_of, widen_tables
    from oracle_drive import table_at
    from paper_2508_08895_amd import binding as A
    wl = W.random_small(seed=6900 + prefix + branches, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2], batch=1,
                        prefix_range=(prefix, prefix), branches_range=(branches, branches), branch_len_range=(1, 9))
    widen_tables(wl, columns)
    gb = GpuBatch(wl)
    gb.grow_to(wl.branch_len)
    tt = table_at(wl, wl.branch_len)
    new = np.ones(wl.NB, dtype=np.int32)
    meta = tt.append_parallel(new)
    step = A.aspd_build_branch_meta(gb.kv, gb.state, A.STAGE_PARALLEL, gb._dev_i32(new), NQ=meta.NQ,
                                    max_new_per_seq=branches if hint else 0)
    q = wl.draw_q(meta.NQ)
    qd, out = q.to(gb.dev), torch.full((meta.NQ, heads[0], heads[2]), float("nan"), dtype=q.dtype, device=gb.dev)

    def call():
        if static:
            A.aspd_attn_parallel_decode_static(gb.kv, gb.state, step, qd, out)
        else:
            A.aspd_attn_parallel_decode(gb.kv, gb.state, step, qd, gb.workspace, out=out)
    call()
    ref, _ = attend(tt, meta, q, wl.k_cache, wl.v_cache)
    assert np.abs(out.float().cpu().numpy() - ref).max() <= TOL
    assert kernels_of(call) == 1


def _chunk_step(heads, batch, prefix, branches, chunk, columns=0, hint=True, cap=0):
    from gpu_drive import GpuBatch, widen_tables
    from oracle_drive import table_at
    from paper_2508_08895_amd import binding as A
    wl = W.random_small(seed=7100 + prefix + chunk, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2], batch=batch,
                        prefix_range=(prefix, prefix), branches_range=(branches, branches), branch_len_range=(1, 1),
                        extra_tokens_per_branch=chunk, extra_tokens_per_seq=0)
    widen_tables(wl, columns)
    gb = GpuBatch(wl)
    gb.grow_to(wl.branch_len)
    tt = table_at(wl, wl.branch_len)
    new = np.full(wl.NB, chunk, dtype=np.int32)
    meta = tt.append_parallel(new)
    step = A.aspd_build_branch_meta(gb.kv, gb.state, A.STAGE_PARALLEL, gb._dev_i32(new), NQ=meta.NQ,
                                    max_new_per_seq=branches * chunk if hint else 0, max_workgroups=cap)
    return wl, gb, tt, meta, step


# On a grid that a table of 1 024 columns leaves whole, an item of one sequence has a part for every sixteen pages or fewer.
@pytest.mark.parametrize("heads,branches,chunk", [((32, 8, 128), 3, 21), ((16, 4, 64), 3, 21), ((2, 2, 128), 4, 60)])
@pytest.mark.parametrize("parts", [1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 16, 17])
def test_every_class_of_parts(heads, branches, chunk, parts):
    """A merge behind the launch in every class of parts, at its first and its last, with as many rows as a row group has or
    nearly: rows in one round and in two, in shares that do not come out even; and with nothing to merge."""
    from gpu_drive import kernels_of, planned_parts, row_splitting_grid
    from paper_2508_08895_amd import binding as A
    wl, gb, tt, meta, step = _chunk_step(heads, 1, 256 * parts - 5 - branches * (chunk + 1), branches, chunk, columns=1024)
    split = planned_parts(step, row_splitting_grid(wl, meta.NQ, branches * chunk))
    assert split == ([parts] * heads[1] if parts > 1 else [])
    q = wl.draw_q(meta.NQ)
    qd = q.to(gb.dev)
    out = torch.full((meta.NQ + 1, *q.shape[1:]), float("nan"), dtype=q.dtype, device=gb.dev)
    lse = torch.full((meta.NQ + 1, heads[0]), float("nan"), dtype=torch.float32, device=gb.dev)

    def call():
        A.aspd_attn_branch_chunk(gb.kv, gb.state, step, qd, gb.workspace, out=out, lse=lse)
    call()
    assert kernels_of(call) == 2
    assert torch.isnan(out[meta.NQ]).all() and torch.isnan(lse[meta.NQ]).all()
    ref, ref_lse = attend(tt, meta, q, wl.k_cache, wl.v_cache)
    assert np.abs(out[:meta.NQ].float().cpu().numpy() - ref).max() <= TOL
    assert np.abs(lse[:meta.NQ].cpu().numpy() - ref_lse).max() <= LSE_TOL


@pytest.mark.parametrize("batch,prefix,branches,chunk,hint,columns,launches", [
    (6, 300, 5, 13, True, 1024, 2),     # 65 rows, a full row group and one query each: 2.7 workgroups an item
    (7, 300, 5, 13, True, 1024, 1),     # 2.3
    (7, 300, 5, 13, False, 1024, 1),    # ... as far as the host can count them without the bound
    (8, 300, 3, 15, True, 1024, 2),     # a row group each: four workgroups an item
    (9, 300, 3, 15, True, 1024, 1),
    (1, 300, 3, 15, False, 1024, 2),
    (1, 300, 3, 15, True, 0, 1),        # a table of the sequence's own width: few workgroups
    (1, 1000, 16, 1, True, 0, 2),
])
def test_where_the_merge_is_a_launch(batch, prefix, branches, chunk, hint, columns, launches):
    """Either side of the lines, and the entry point without a workspace where its scratch is enough."""
    from gpu_drive import kernels_of
    from paper_2508_08895_amd import binding as A
    wl, gb, tt, meta, step = _chunk_step((32, 8, 128), batch, prefix, branches, chunk, columns, hint)
    q = wl.draw_q(meta.NQ)
    qd = q.to(gb.dev)
    calls = [lambda out: A.aspd_attn_branch_chunk(gb.kv, gb.state, step, qd, gb.workspace, out=out)]
    if chunk == 1:
        calls.append(lambda out: A.aspd_attn_parallel_decode_static(gb.kv, gb.state, step, qd, out))
    ref, _ = attend(tt, meta, q, wl.k_cache, wl.v_cache)
    for call in calls:
        out = torch.full_like(qd, float("nan"))
        call(out)
        assert np.abs(out.float().cpu().numpy() - ref).max() <= TOL
        # (a step without the bound has its plan built for decoding: the chunk call works one out itself)
        assert kernels_of(lambda: call(out)) == launches + (0 if hint else 1)


@pytest.mark.parametrize("heads,cap", [((6, 3, 128), 2), ((12, 6, 128), 5), ((16, 16, 128), 9), ((32, 8, 128), 40), ((4, 1, 64), 3)])
def test_row_groups_sequence_by_sequence(heads, cap):
    """More tokens than an L2 holds of one KV head: the list goes sequence by sequence, longest first and in each longest ranges
    first, and holds every row group once; sequences of equal and of different length, with parallel stages and without, one
    empty; odd numbers of heads, and more heads than queues."""
    from gpu_drive import GpuBatch
    from paper_2508_08895_amd import binding as A
    G, D = heads[0] // heads[1], heads[2]
    qpg, l2 = 256 // G, (4 << 20) // (4 * D)                 # tokens of a row group, and of one KV head in an L2
    n = l2 // 4 + 57
    layouts = [[(0, n // 3), (1, 40), (2, n // 3), (3, 7), (0, n - 2 * (n // 3) - 47)], [(0, 5)], [],
               [(0, n)], [(0, 100), (1, n // 2), (2, n - n // 2 - 100)], [(0, n + qpg)]]
    lengths = [sum(m for _, m in r) for r in layouts]
    wl = W.random_small(seed=7300 + heads[0], num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=D, batch=len(layouts),
                        prefix_range=(max(lengths), max(lengths)), branches_range=(1, 1), branch_len_range=(1, 1))
    tt, meta = replay_layout(wl.block_tables, wl.block_size, layouts)
    gb = GpuBatch(wl)
    step = A.aspd_build_sequence_meta(gb.kv, gb.state, gb._dev_i32(np.cumsum([0] + [len(r) for r in layouts])),
                                      gb._dev_i32([b for r in layouts for b, _ in r]),
                                      gb._dev_i32([m for r in layouts for _, m in r]), NQ=meta.NQ, max_workgroups=cap)
    words = step.plan.view(torch.int32).cpu().numpy()
    items = words[0]
    assert items == sum(-(-m // qpg) for m in lengths) and items * qpg > l2 and items * heads[1] >= 12 * cap
    first = np.cumsum([0] + lengths)
    want = [(s, first[s] + t, min(qpg, lengths[s] - t), (min(t + qpg, lengths[s]) + 15) // 16)
            for s in sorted(range(len(lengths)), key=lambda s: (-(-(-lengths[s] // qpg)), s))
            for t in reversed(range(0, lengths[s], qpg))]
    at = 16 + (meta.NQ + 3) // 4 * 4
    assert words[at:at + 4 * items].reshape(items, 4).tolist() == [list(map(int, w)) for w in want]
    q = wl.draw_q(meta.NQ)
    out = torch.full(q.shape, float("nan"), dtype=q.dtype, device=gb.dev)
    A.aspd_attn_full_sequence(gb.kv, gb.state, step, q.to(gb.dev), gb.workspace, out=out)
    assert torch.isfinite(out).all()
    assert int(gb.workspace[:4096].view(torch.int32).abs().sum().item()) == 0
    rows = sorted({*range(0, meta.NQ, 331), *(int(x) - 1 for x in first[1:]), *(int(x) for x in first[:-1] if x < meta.NQ)})
    ref, _ = attend(tt, meta, q, wl.k_cache, wl.v_cache, rows=rows)
    assert np.abs(out.float().cpu().numpy()[rows] - ref[rows]).max() <= TOL

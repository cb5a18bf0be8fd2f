"""The metadata call on steps that it refuses in part: the plan stays inside its buffer and names rows of the step only."""
import numpy as np
import pytest
import torch

from paper_2508_08895_amd import binding as A

pytestmark = pytest.mark.gpu

_GUARD = 0x5a5a5a5a


def _batch(B, count, max_blocks=24):
    pool = torch.zeros(B * max_blocks, 2, 16, 64, dtype=torch.bfloat16, device="cuda")
    tables = torch.arange(B * max_blocks, dtype=torch.int32).reshape(B, max_blocks).cuda()
    kv = A.KVCache(pool, pool, tables, 8)
    st = A.BatchState(B, max_blocks * 16, "cuda")
    st.cu_branches = torch.from_numpy(np.append(0, np.cumsum(count)).astype(np.int32)).cuda()
    st.NB = int(sum(count))
    st.branch_len = torch.zeros(st.NB, dtype=torch.int32, device="cuda")
    st.stage_base.fill_(100)
    st.seq_len.fill_(100)
    return kv, st


@pytest.mark.parametrize("B", [1, 3, 64, 500])
@pytest.mark.parametrize("hint", [0, 7, 60])   # streaming kernel without and with a hint, row-splitting kernel
@pytest.mark.parametrize("kind", ["main tokens under open branches", "more tokens than rows"])
def test_plan_of_a_refused_step_stays_in_its_buffer(B, hint, kind):
    count = np.where(np.arange(B) % 2 == 0, 2, 0)
    kv, st = _batch(B, count)
    main = np.full(B, 3)
    if kind == "more tokens than rows":
        main[count > 0] = 0
    new = np.full(st.NB, 2)
    rows = int(new.sum() + main.sum()) if kind != "more tokens than rows" else 5
    step = A.Step(rows, st.NB, B, "cuda", max_new_per_seq=hint)
    step.cu_seq_new.copy_((torch.arange(B + 1) % 2 * 4000).int())   # as earlier steps may have left them
    words = A.aspd_plan_bytes(kv, B, rows) // 4
    whole = torch.full((words + 4096,), _GUARD, dtype=torch.int32, device="cuda")
    step.plan = whole[:words]
    lens = torch.from_numpy(np.concatenate([new, main]).astype(np.int32)).cuda()
    A.aspd_build_branch_meta(kv, st, A.STAGE_MIXED, lens, step=step)
    assert bool((whole[words:] == _GUARD).all())
    fault = int(st.fault[0])
    assert fault & (A.FAULT_ROW_COUNT if kind == "more tokens than rows" else A.FAULT_STAGE) or (B == 1 and rows == 5)
    # every sequence's rows begin where those before it end, refused or not
    per_seq = np.add.reduceat(np.append(new, 0), np.append(0, np.cumsum(count))[:-1]) * (count > 0) + main
    assert np.array_equal(step.cu_seq_new.cpu().numpy(), np.append(0, np.cumsum(per_seq)))
    # no segment of the plan names a row that the step does not have
    plan = step.plan.cpu().numpy()
    nwg = step.plan_key >> 27 & 2047
    for w in range(nwg):
        n, at = plan[32 * w + 8], plan[32 * w + 9]
        segs = [plan[32 * w:32 * w + 8]] if n > 0 else []
        segs += [plan[32 * nwg + 8 * (at + i):32 * nwg + 8 * (at + i + 1)] for i in range(n - 1)]
        for d in segs:
            assert 0 <= d[1] and 1 <= d[2] and d[1] + d[2] <= rows, (w, d)

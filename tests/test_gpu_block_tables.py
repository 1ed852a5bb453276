"""The block-table compaction at its edges: groups of 64 ids, batches of table
entries, and pools of one window of 65536 ids, just past it and two windows
with free ids, three whole ones and a ragged fourth (the list of live ids then
grows up to the flags in memory), and tables that are mostly unused slots, out of place (positions in the live list) and in place (block
ranges resolved by rank), against the oracle; ids out of range and a wrong
live count in the last window are refused.  GPU, through the C ABI."""
import numpy as np
import pytest
import torch

from paper_2511_11617_amd import atp, problem
from synth import configs
from synth.content import KIND_RAW16
from tests.gpu_harness import run_case

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _cfg(n_seq, per_seq, factor):
    # blocks of one token, 32-byte heads, one layer; KV heads 1 -> 2 on this rank (a chain of levels in place)
    return configs.get(1, layers=1, n_q=8, n_kv=4, head_dim=16, block_tokens=1, n_seq=n_seq, seq_tokens=per_seq,
                       new_q_widths=None, self_old=2, fragmented=factor > 1.0, pool_factor=factor,
                       w_kind=KIND_RAW16, kv_kind=KIND_RAW16)


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("n_seq,per_seq,factor", [
    (1, 1, 1.0), (3, 21, 1.0), (1, 64, 1.5), (5, 13, 1.0), (1, 1024, 1.0), (1, 1025, 1.1), (4, 1024, 1.0),
    (3, 1367, 1.3), (8, 1024, 1.0), (3, 2731, 1.0), (16, 1024, 1.25), (5, 3277, 1.0), (16, 4096, 1.0),
    (16, 4097, 1.0), (16, 4096, 2.01), (48, 4096, 1.0), (7, 28101, 1.0), (7, 28101, 1.3)])
def test_pool_and_table_sizes(n_seq, per_seq, factor, inplace):
    run_case(_cfg(n_seq, per_seq, factor), flags=atp.INPLACE if inplace else 0,
             name=f"table-{n_seq}x{per_seq}-{factor}")


@pytest.mark.parametrize("pool,slots", [(65536, 300000), (65537, 300000), (200001, 1 << 20)])
def test_sparse_tables(pool, slots):
    """Most slots unused (-1 and other negative numbers), ids repeated and in any
    order: only the pool's live blocks move."""
    rng = np.random.default_rng(pool)
    c = _cfg(1, pool, 1.0)
    ids = rng.permutation(pool)[:pool // 3].astype(np.int32)
    plan = problem.build(c, n_live=ids.size, pool=pool).plan()
    st = plan.stats()
    table = rng.choice(np.array([-1, -2, -65536, -2 ** 31], np.int32), slots)
    at = rng.permutation(slots)[:ids.size + 1000]
    table[at] = np.concatenate([ids, ids[:1000]])
    dev = torch.device("cuda")
    old = torch.from_numpy(rng.integers(0, 256, st.old_kv_bytes, dtype=np.uint8)).to(dev)
    new = torch.full((st.new_kv_bytes,), 0xA5, dtype=torch.uint8, device=dev)
    hin_np = rng.integers(0, 256, st.inflow_kv, dtype=np.uint8)
    hin = torch.empty(max(1, st.inflow_kv), dtype=torch.uint8, pin_memory=True)
    hin[:st.inflow_kv].copy_(torch.from_numpy(hin_np))
    stage = torch.zeros(st.staging_kv, dtype=torch.uint8, device=dev)
    td = torch.from_numpy(table).to(dev)
    copy = torch.cuda.Stream()
    torch.cuda.synchronize()
    plan.reshard_kv(old.data_ptr(), old.numel(), new.data_ptr(), new.numel(), td.data_ptr(), 1, slots, hin.data_ptr(),
                    st.inflow_kv, None, 0, stage.data_ptr(), stage.numel(),
                    torch.cuda.current_stream().cuda_stream, copy.cuda_stream)
    plan.sync()
    torch.cuda.synchronize()
    # 32-byte heads of one-token blocks: the old shard's heads are the first or last of the new one's
    heads_old, heads_new = st.old_kv_bytes // (2 * pool * 32), st.new_kv_bytes // (2 * pool * 32)
    (o0, o1), (n0, n1) = plan.old_ranges(1)[c["self_old"]], plan.ranges(1)[st.self_new_rank]
    assert (o1 - o0, n1 - n0) == (heads_old, heads_new) and n0 <= o0 and o1 <= n1
    live = np.sort(ids)
    want = np.full((2, pool, heads_new, 32), 0xA5, np.uint8)
    want[:, live, o0 - n0:o1 - n0] = old.cpu().numpy().reshape(2, pool, heads_old, 32)[:, live]
    for sg in plan.segments(atp.SEG_INFLOW_KV):
        part = hin_np[sg.host_offset:sg.host_offset + sg.bytes].reshape(live.size, -1, 32)
        want[sg.which, live, sg.unit_begin - n0:sg.unit_end - n0] = part
    np.testing.assert_array_equal(new.cpu().numpy().reshape(want.shape), want)


@pytest.mark.parametrize("fault", ["id", "count"])
def test_bad_entry_in_the_second_window_moves_nothing(fault):
    n, pool = 70000, 70016
    c = _cfg(1, n, 1.0)
    b = problem.build(c, n_live=n, pool=pool)
    plan = b.plan()
    st = plan.stats()
    table = np.arange(n, dtype=np.int32)
    table[66000] = pool if fault == "id" else table[66001]
    dev = torch.device("cuda")
    old = torch.zeros(st.old_kv_bytes, dtype=torch.uint8, device=dev)
    new = torch.full((st.new_kv_bytes,), 0xA5, dtype=torch.uint8, device=dev)
    hin = torch.zeros(st.inflow_kv, dtype=torch.uint8, pin_memory=True)
    stage = torch.zeros(st.staging_kv, dtype=torch.uint8, device=dev)
    td = torch.from_numpy(table).to(dev)
    copy = torch.cuda.Stream()
    torch.cuda.synchronize()
    plan.reshard_kv(old.data_ptr(), old.numel(), new.data_ptr(), new.numel(), td.data_ptr(), 1, n, hin.data_ptr(),
                    st.inflow_kv, None, 0, stage.data_ptr(), stage.numel(),
                    torch.cuda.current_stream().cuda_stream, copy.cuda_stream)
    with pytest.raises(atp.AtpError) as e:
        plan.sync()
    assert e.value.code == atp.EINVAL and ("num_blocks" if fault == "id" else "live blocks") in str(e.value)
    torch.cuda.synchronize()
    assert bool((new == 0xA5).all())

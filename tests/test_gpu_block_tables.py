"""The block-table compaction at its edges: groups of 64 ids, batches of table
entries, and pools of one window of 65536 ids, just past it and two windows
with free ids, out of place (positions in the live list) and in place (block
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
    (16, 4097, 1.0), (16, 4096, 2.01)])
def test_pool_and_table_sizes(n_seq, per_seq, factor, inplace):
    run_case(_cfg(n_seq, per_seq, factor), flags=atp.INPLACE if inplace else 0,
             name=f"table-{n_seq}x{per_seq}-{factor}")


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

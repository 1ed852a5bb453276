"""Lines that are not 16-byte aligned, at the sizes where the copy kernel's
chunks change: runs shorter than one chunk, one chunk and a byte more or
less, a tile of chunks and one more or less, for element sizes of 1, 2 and 3
bytes and every misalignment a row pitch gives, out of place and in place
(host reads, repack and outbound reads); and aligned columns at the edges of
the link kernel's tiles.  Expected bytes are slices of the full matrix.  GPU, through the C ABI."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2511_11617_amd import atp
from synth import configs
from synth.content import KIND_RAW16
from tests.gpu_harness import run_case, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _problem(rows, old_w, new_w, eb, flags):
    """One row-parallel [rows, sum(old_w)] matrix, TP 3 -> 2, rank 0 failed,
    this GPU old rank 1 (new rank 0)."""
    sp = atp.Space()
    sp.total_units, sp.old_tp, sp.new_tp = sum(old_w), 3, 2
    keep = [(C.c_int64 * 3)(*old_w), (C.c_int64 * 2)(*new_w)]
    sp.old_rule = sp.new_rule = atp.RULE_WIDTHS
    sp.old_widths, sp.new_widths = (C.cast(k, C.POINTER(C.c_int64)) for k in keep)
    t = atp.Tensor()
    t.space, t.kind, t.layer, t.elem_bytes = 0, atp.COLS, 0, eb
    t.rows, t.cols, t.unit, t.old_offset = rows, sum(old_w), 1, atp.OFFSET_AUTO
    failed = (C.c_int32 * 1)(0)
    pb = atp.Problem()
    pb.n_spaces, pb.n_tensors, pb.n_failed = 1, 1, 1
    pb.spaces, pb.tensors = C.pointer(sp), C.pointer(t)
    pb.failed = C.cast(failed, C.POINTER(C.c_int32))
    pb.self_old_rank, pb.flags = 1, flags
    return atp.Plan(pb, keep=(keep, sp, t, failed))


def check_columns(rows, old_w, new_w, eb, inplace, seed):
    say(f"[columns] rows={rows} eb={eb} inplace={inplace} widths={old_w}->{new_w}")
    plan = _problem(rows, old_w, new_w, eb, atp.INPLACE if inplace else 0)
    st = plan.stats()
    full = np.random.default_rng(seed).integers(0, 256, (rows, sum(old_w), eb), dtype=np.uint8)
    part = lambda a, b: np.ascontiguousarray(full[:, a:b]).reshape(-1)
    old, want = part(old_w[0], old_w[0] + old_w[1]), part(0, new_w[0])
    hosts = []
    for which, n in ((atp.SEG_INFLOW_W, st.inflow_w), (atp.SEG_OUTBOUND_W, st.outbound_w)):
        h = np.zeros(n, np.uint8)
        for s in plan.segments(which):
            h[s.host_offset:s.host_offset + s.bytes] = part(s.unit_begin, s.unit_end)
        hosts.append(h)
    size = max(st.old_arena_bytes, st.new_arena_bytes)
    a = torch.full((size + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    a[:old.size].copy_(torch.from_numpy(old))
    n = a if inplace else torch.full((size + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    hin = torch.empty(max(hosts[0].size, 1), dtype=torch.uint8, pin_memory=True)
    hin[:hosts[0].size].copy_(torch.from_numpy(hosts[0]))
    hout = torch.full((hosts[1].size + 64,), 0x3C, dtype=torch.uint8, pin_memory=True)
    stage = torch.empty(max(st.staging_w, 256), dtype=torch.uint8, device="cuda")
    s1 = torch.cuda.Stream()
    torch.cuda.synchronize()
    plan.reshard_weights(a.data_ptr(), size, None if inplace else n.data_ptr(), 0 if inplace else size,
                         hin.data_ptr(), st.inflow_w, hout.data_ptr(), st.outbound_w if inplace else 0,
                         stage.data_ptr(), stage.numel(), torch.cuda.current_stream().cuda_stream,
                         s1.cuda_stream)
    plan.sync()
    torch.cuda.synchronize()
    got = n.cpu().numpy()
    np.testing.assert_array_equal(got[:want.size], want)
    assert (got[max(want.size, old.size if inplace else 0):] == 0xA5).all()  # nothing past the shard
    if inplace:
        np.testing.assert_array_equal(hout.numpy()[:hosts[1].size], hosts[1])
        assert (hout.numpy()[hosts[1].size:] == 0x3C).all()


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("eb", [1, 2, 3])
@pytest.mark.parametrize("run", [1, 5, 7, 15, 16, 17, 31, 33, 511, 8175, 8193, 16385])
def test_ragged_columns(run, eb, inplace):
    # old ranks hold a, b, c columns; new rank 0 takes all but the last d:
    # its inflow is a columns, it keeps b of its own, or drops some of them
    rows = 37 if run > 1000 else 1021
    for old_w, new_w in (((run, run + 1, 3), (2 * run + 1, 3)),   # keeps all, shifted by its inflow
                         ((3, run + 4, run), (run + 3, run + 4))):  # drops the last ones to its peer
        check_columns(rows, old_w, new_w, eb, inplace, run * 4 + eb)


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("rows", [511, 512, 513])
@pytest.mark.parametrize("tiles", [1, 19, 20, 21, 40, 41, 60, 61])
def test_link_tiles(tiles, rows, inplace):
    """Aligned columns (16-byte elements) whose host read, or outbound read,
    takes `tiles` tiles of 512 chunks, a chunk row more or less: fewer than
    the workgroups, one each, and odd and even numbers in flight."""
    keep = 16 * tiles + 1  # a repack long enough for two tiles in flight per workgroup
    check_columns(rows, (tiles, keep, 3), (tiles + keep, 3), 16, inplace, tiles)
    check_columns(rows, (1, keep + tiles, 3), (1 + keep, tiles + 3), 16, inplace, tiles)


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("layout", ["head", "token"])
@pytest.mark.parametrize("head_dim", [3, 7, 9, 20])
def test_ragged_kv_heads(head_dim, layout, inplace):
    c = configs.get(1, head_dim=head_dim, kv_layout=layout, block_tokens=5, seq_tokens=125, n_q=8, n_kv=4,
                    new_q_widths=None, w_kind=KIND_RAW16, kv_kind=KIND_RAW16, self_old=2)
    run_case(c, flags=atp.INPLACE if inplace else 0, name=f"ragged-kv-{head_dim}-{layout}")

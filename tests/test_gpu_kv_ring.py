"""The in-place KV inflow chunk by chunk: read by the copy kernel from a
pinned inflow buffer into place or, where it would wait for late levels,
into its slot, and through the landing ring from pageable memory or a
buffer the kernel cannot read (not 256-byte aligned), with chunks of one and
of several copies, against the oracle.  GPU, through the C ABI."""
import numpy as np
import pytest
import torch

from paper_2511_11617_amd import atp
from synth import configs
from synth.content import KIND_RAW16
from tests.gpu_harness import SQUEEZED_RING_CAP, late_gates_cfg, squeezed_ring_cfg
from tests.test_zz_no_alloc import _KV

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _ragged(head_dim):
    # pieces of odd sizes: a chunk takes several copies, each at a 256-byte boundary of its slot
    return configs.get(1, layers=3, n_q=8, n_kv=4, head_dim=head_dim, block_tokens=5, seq_tokens=125, n_seq=9,
                       new_q_widths=None, self_old=2, w_kind=KIND_RAW16, kv_kind=KIND_RAW16)


@pytest.mark.parametrize("memory", ["pinned", "pageable", "misaligned"])
@pytest.mark.parametrize("name", ["ring-of-16-chunks", "odd-pieces", "one-odd-head", "late-gates",
                                  "late-gates-last-tile", "late-gates-four-slots", "outbound-beside", "wide-lines"])
def test_in_place_kv_inflow(name, memory):
    cfg, cap = {"ring-of-16-chunks": (squeezed_ring_cfg(), SQUEEZED_RING_CAP),
                "odd-pieces": (_ragged(7), 1 << 30),
                "one-odd-head": (dict(_ragged(20), layers=1), 1 << 30),
                "late-gates": (late_gates_cfg(), 1 << 30),
                "late-gates-last-tile": (late_gates_cfg(head_dim=12), 1 << 30),  # not whole tiles of 8 KiB
                "outbound-beside": (late_gates_cfg(n_q=16, n_kv=8, head_dim=80, layers=4, n_seq=4, seq_tokens=2048,
                                                   fragmented=False, pool_factor=1.0, block_tokens=16,
                                                   new_kv_widths=[4, 4], kv_rule="widths"), 1 << 30),
                "late-gates-four-slots": (late_gates_cfg(layers=2), 24 << 20),
                "wide-lines": (configs.scaled(5, layers=2, n_seq=2, seq_tokens=1024, kv_kind=KIND_RAW16),
                               1 << 30)}[name]
    k = _KV(cfg, atp.INPLACE, staging_cap=cap)
    assert k.inflow.size > 0
    if memory == "pageable":
        k.hin = torch.from_numpy(np.concatenate([k.inflow, np.zeros(1, np.uint8)]))
    elif memory == "misaligned":
        t = torch.empty(k.inflow.size + 64, dtype=torch.uint8, pin_memory=True)
        k.hin = t[64:]
        k.hin.copy_(torch.from_numpy(k.inflow))
    streams = torch.cuda.current_stream(), torch.cuda.Stream()
    got, out = k.run(False, streams)
    bad = np.flatnonzero(got[k.mask] != k.want[k.mask])
    assert bad.size == 0, f"{bad.size} live bytes differ from the oracle, first at {bad[:5]}"
    np.testing.assert_array_equal(out, k.outbound)

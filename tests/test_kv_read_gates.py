"""The in-place KV inflow read straight from the host buffer beside the
levels: every read as early as its gate allows, replayed on the host against
the oracle (the replay finds a level that reads bytes a read already landed
on, and wrong places).  CPU."""
import random

import pytest

from paper_2511_11617_amd import atp
from synth import configs
from synth.content import KIND_TAG16
from tests.gpu_harness import SQUEEZED_RING_CAP, squeezed_ring_cfg
from tests.schedule_sim import H2D, H2D_RING, INFLOW, SCATTER, Hazard
from tests.test_oracle_repack import med_cfg, tiny_cfg
from tests.test_schedule_sim import _clone, sim_case


def _reads(early=0, seen=None):
    """Each slot's scatters as landings from the inflow buffer, `early` levels
    before their gates."""
    def change(which, cps):
        if which == 0:
            return cps
        out, ring = [], []
        for i, x in enumerate(cps):
            if x.op == H2D_RING:
                ring = ring + [x] if cps[i - 1].op == H2D_RING else [x]
            if x.op == SCATTER and len(ring) == 1:
                if seen is not None:
                    seen.append(x.level)
                out.append(_clone(x, op=H2D, src_buf=INFLOW, level=max(-1, x.level - early),
                                  src_off=x.src_off - ring[0].dst_off + ring[0].src_off))
                if ring[0] in out:
                    out.remove(ring[0])
            else:
                out.append(x)
        return out
    return change


def _chain(**kw):
    return configs.get(5, layers=4, hidden=512, n_q=16, n_kv=8, head_dim=64, ffn=1024, n_seq=8, seq_tokens=4096,
                       new_q_widths=None, w_kind=KIND_TAG16, kv_kind=KIND_TAG16, **kw)


@pytest.mark.parametrize("no_tail", [False, True])
def test_chain_of_levels(no_tail):
    seen = []
    sim_case(_chain(), flags=atp.INPLACE | (atp.NO_TAIL_STAGING if no_tail else 0), mutate=_reads(seen=seen))
    # the upper planes at once, the lower ones after a level
    assert min(seen) == -1 and max(seen) >= int(no_tail)


def test_read_before_its_gate_is_caught():
    with pytest.raises((Hazard, AssertionError)):
        sim_case(_chain(), flags=atp.INPLACE | atp.NO_TAIL_STAGING, mutate=_reads(early=100))


def test_many_chunks():
    sim_case(squeezed_ring_cfg(), flags=atp.INPLACE, staging_cap=SQUEEZED_RING_CAP, mutate=_reads())


@pytest.mark.parametrize("seed", range(30))
def test_random_small(seed):
    c = tiny_cfg(random.Random(7000 + seed), seed % 3 == 0)
    sim_case(c, flags=atp.INPLACE | (atp.NO_TAIL_STAGING if seed % 2 else 0), mutate=_reads())


@pytest.mark.parametrize("seed", range(6))
def test_random_medium(seed):
    sim_case(med_cfg(random.Random(8000 + seed), experts=seed % 3 == 0), flags=atp.INPLACE, mutate=_reads())

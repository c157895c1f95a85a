"""Where a call takes one kernel or another, by its size: the results on both
sides of each line, and against references that do not depend on it."""
import numpy as np
import pytest
import torch

import oracle
from paper_2106_13281_amd import braxmi, synth
from test_gpu_split import SYSTEMS, equal, head, inputs

pytestmark = pytest.mark.gpu


def n_cu():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("E", [50, 9000])  # two wavefronts per work item, one
def test_control_cost_rounding(E):
    """A three-axis joint's squared actions are added by fused multiply-adds in axis
    order and the bodies' in body order, on every kernel: exact (tolerance zero)."""
    name = "biped"
    o = oracle.Oracle(synth.system_text(name)).system
    s = braxmi.System(synth.system_text(name), E, device=0)
    x, acts = inputs(s, 4, 1)
    a = acts[0].contiguous()
    s.env_configure([dict(forward_weight=0.0, healthy_reward=0.0, ctrl_cost=1.0)])
    _, _, reward, _ = s.env_step(x, a, s.default_qp())
    a = a.cpu().numpy()
    ctrl = np.zeros(E, np.float32)
    for b in range(o.nb):
        sq = np.zeros(E, np.float32)
        for k, act in enumerate(o.actions):
            if o.joints[act[0]]["child"] == b:
                r = a[k].astype(np.longdouble)
                sq = (r * r + sq).astype(np.float32)
        ctrl += sq
    assert np.array_equal(reward.cpu().numpy(), -ctrl)

"""Layer-by-layer parity (tests/layerwise.py, bars of tests/test_gpu_layerwise.py) of small modules whose shapes sit at the
edges of the rules that choose a kernel: partly filled channel groups, remainders of tiles, the ends of a rule's range."""
import pytest

import fdg_workloads as W
from fdg_workloads import Layer, ModuleSpec
from tests import test_gpu_layerwise as LT

pytestmark = pytest.mark.gpu

H = dict(momentum=0.9, weight_decay=5e-4, bn_eps=1e-5, bn_momentum=0.1, lr=0.01)


def check(name, spec):
    print(f"case {name} layer by layer", flush=True)
    plain = []
    LT._judge(LT._run(spec, seed=1, steps_after_warmup=2, plain=plain), name)
    LT._judge_plain(plain, name)


# A module with narrow 3x3 kernels keeps its batch-norm sums in eight copies, which the batch-norm kernels fold by workgroup:
# 1, 2, 4 and 8 channel groups a workgroup, one of them partly filled (24, 40 and 72 channels), one and two normalised operands
COPIES = {
    "copies preact": [Layer(W.BASIC_PREACT, 16, 16, 1), Layer(W.BASIC_PREACT, 16, 24, 1), Layer(W.BASIC_PREACT, 24, 8, 1),
                      Layer(W.BASIC_PREACT, 8, 72, 1)],
    "copies postact": [Layer(W.BASIC_POSTACT, 16, 40, 2), Layer(W.BASIC_POSTACT, 40, 8, 1), Layer(W.BASIC_POSTACT, 8, 72, 1),
                       Layer(W.BASIC_POSTACT, 72, 16, 1), Layer(W.BASIC_POSTACT, 16, 16, 1)],
}


@pytest.mark.parametrize("name", sorted(COPIES))
def test_sums_in_copies(name):
    check(name, ModuleSpec(6, 16, 23, 21, COPIES[name], delay=1, is_bottom=False, beta=0.5, name=name, **H))

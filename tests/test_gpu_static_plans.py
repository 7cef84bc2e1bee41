"""xm_count_static with about as many plans as its array can hold: 22,518 plans of
one enumerated level filled it to within 512 bytes when the launch kept 512 KiB
of donated-task slots, and must go on being accepted."""
import pytest

import oracle
import xmgen
from tests.test_zz_no_alloc import static_count

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 5000, 22518])
def test_many_plans_fit_the_static_array(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_11105_amd as xa
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the figure is for 256 compute units")
    g = xmgen.complete_digraph(5)
    G = xa.Graph(g)
    p = xmgen.named("arc")
    plan = xa.Plan(p, graph=G)
    assert plan.describe()["e"] == 1
    print("[case]", n, flush=True)
    got, status = static_count(xa, G, [plan] * n)
    assert status == [0] * n and got == [oracle.count(g, p)] * n

"""A lattice may be released after its context, as Python's garbage collector does with both in one cycle."""
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_0910_1048_amd as sgn  # noqa: E402
from gpu_util import dev  # noqa: E402


def test_a_lattice_outlives_its_context():
    dims = (16, 16, 16, 16)   # 6 rows of links in three precisions: 44 MB
    U = dev(synth.gauge_field(dims, 0.4, 1))
    keep = [sgn.Context(0) for _ in range(3)]   # later contexts may take the released one's memory
    c = sgn.Context(0)
    lat = sgn.Lattice(c, U, dims)
    torch.cuda.synchronize()
    held, _ = torch.cuda.mem_get_info()
    c.close()
    del keep
    lat.close()   # raises if the device cannot be told
    freed, _ = torch.cuda.mem_get_info()
    assert freed - held >= 30 << 20

"""The long max-convolution on a workspace sized for another family: fewer p
at a time give the same bits (every p is transformed by itself); below two p
the call is refused."""

import pytest

from workloads import maxconv_vectors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,n,m", [(48, 6001, 3500), (80, 2100, 2003), (3, 8192, 8193)])
@pytest.mark.parametrize("sized_for", [[8], [1, 2, 4, 8, 16, 32, 64]], ids=["one", "seven"])
def test_workspace_of_another_family(gpu_lib, b, n, m, sized_for):
    import torch

    mt = gpu_lib
    P = list(range(1, 25))
    x, y = (torch.from_numpy(v).cuda() for v in maxconv_vectors(b, n, m, 5, "uniform"))
    print(f"[maxconv] {b} x {n}, {m} workspace of {len(sized_for)} p", flush=True)
    size = mt.maxconv_workspace_size(b, n, m, sized_for)
    full = mt.maxconv_workspace_size(b, n, m, P)
    assert size <= full
    z0, ps0 = mt.maxconv(x, y, P, return_pstar=True)
    ws = torch.full((size + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    z, ps = mt.maxconv(x, y, P, return_pstar=True, workspace=ws[:size])
    assert torch.equal(z, z0) and torch.equal(ps, ps0)
    assert bool((ws[size:] == 0xFF).all())
    least = mt.maxconv_workspace_size(b, n, m, [8])
    with pytest.raises(mt.MaxTimesError) as e:
        mt.maxconv(x, y, P, workspace=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))
    assert e.value.status == 3

"""What the autotuner reports for a lattice march, and decides by, is the time of a step that its launches took: a
patch launch of 24 or 8 steps takes only those that are left of 12, rounded up to four."""
import numpy as np
import pytest

import paper_1705_01387_amd as P
from paper_1705_01387_amd import inputs as I

pytestmark = pytest.mark.gpu
CASES = {      # steps of the launches that 12 recurrence steps take
    "chain": (lambda: I.chain(3_000_000, W=1.0, seed=1), 1, 12),
    "square_patches": (lambda: I.square(176, 160, W=1.0, seed=2), 4, 12),
    "square_march": (lambda: I.square(1400, 1300, W=1.0, seed=3), 1, 16),
}


@pytest.mark.parametrize("name", list(CASES))
def test_march_time_is_per_step(gpu, name):
    """Against events around the same 12 steps: a division by 24 or 16 made it half and three quarters."""
    import torch
    print(f"case: march time {name}", flush=True)
    make, B, taken = CASES[name]
    m = make()
    H = P.gpuqt_build_h_from_model(m)
    code = H.info.kernel_variant
    got = min(P.gpuqt_autotune(H, B)[6] for _ in range(3))
    P.gpuqt_set_variant(H, code)
    d = torch.from_numpy(I.random_phase(m.n, B, 4)).cuda()
    ws = torch.empty(P.gpuqt_workspace_size(H, P.OP_MOMENTS, B, 24), dtype=torch.uint8, device="cuda")
    P.gpuqt_set_timing(H, True)
    us = []
    for _ in range(6):
        P.gpuqt_timing(H)
        P.gpuqt_moments(H, d, d, 24, ws=ws)
        ms, launches = P.gpuqt_timing(H)["moment_sym"]
        us.append(1e3 * ms / taken)
    assert launches < 12
    assert 0.8 * min(us) < got < 1.5 * min(us), (got, us)

"""Kernel variants and dispatch edges on the GPU, each against the float64 oracle."""
import numpy as np
import pytest

import oracle as O
from harness import dev_bf16, host_f32
from workloads import BlockShape, make_rng
from workloads.gen import draw_time_weights

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A(gpu):
    from paper_2606_15319_amd import ardit
    return ardit


def _sync():
    import torch
    torch.cuda.synchronize()


@pytest.mark.parametrize("dim,n", [(128, 1), (640, 2), (1152, 9), (2816, 3), (2816, 8)])
def test_time_mod_rows_and_stream_groups(A, dim, n):
    """Rows per wave (four from 16384 outputs: 6 x 2816 = 16896), streams in
    groups of eight, and widths that end inside a 512- or 1024-column step."""
    import torch
    tw = draw_time_weights(make_rng(400), dim)
    ts = [100.0 * i + 37.5 for i in range(n)]   # exact in fp32 (an angle is t times up to 1 rad)
    sh = BlockShape(dim=dim, n_heads=dim // 128, head_dim=128, ffn_dim=128, frames=1, lat_h=8, lat_w=8)
    mod = torch.full((n, 6, dim), float("nan"), device="cuda")
    ws = torch.empty(4 << 20, dtype=torch.uint8, device="cuda")
    A.ardit_time_mod(None, A.dims_from_shape(sh), ts,
                     A.time_weights({k: dev_bf16(v) for k, v in tw.items()}), mod, ws, ws.numel())
    _sync()
    got = host_f32(mod)
    for i, t in enumerate(ts):
        ref = O.time_modulation(t, tw, dim)
        # three chained fp32 sums of K <= 2816 terms: a sum's rounding error is a
        # random walk of about sqrt(K) 2^-24 of its RMS, 3.2e-6; three of them
        # and a factor of two for the largest of 17k values: 2e-5 of the RMS
        assert np.max(np.abs(got[i] - ref)) <= 2e-5 * np.sqrt(np.mean(ref ** 2)), (dim, n, i)

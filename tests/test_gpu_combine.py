"""The merge of an encode's split-key partials through the routing entry
point: values that are not finite, against what the softmax defines for them
(a zero weight times an infinity or a NaN is a NaN).
"""

import numpy as np
import pytest
import torch

from paper_2608_11519_amd import flarepp as fp
from paper_2608_11519_amd import inputs as inp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fp.load()
    yield


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [16, 32, 64])
def test_non_finite_value_in_a_chunk_without_weight(monkeypatch, D, dtype, bad):
    # eight chunks of 128 tokens; the scores of chunk 3 are +400 (natural log
    # units), those of the others -400, so the others' weight is exactly zero
    # in fp32.  One value in chunk 7 is not finite: 0 * bad is a NaN in its
    # channel of every route, and every other channel is the mean of chunk 3.
    # (chunks 3 and 7 meet in one thread's fold at every D)
    monkeypatch.setenv("FLAREPP_FORCE_CHUNKS", "8")
    N, M, bad_n, bad_d = 1024, 20, 928, 5
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    q = torch.full((1, 1, M, D), 20.0, device="cuda")
    k = torch.full((1, 1, N, D), -20.0 / D ** 0.5, device="cuda")
    k[:, :, 3 * 128:4 * 128] *= -1
    v = torch.from_numpy(inp.make_tensor((1, 1, N, D), 41, dtype)).cuda()
    want = v[0, 0, 3 * 128:4 * 128].double().mean(0).cpu().numpy()
    v[0, 0, bad_n, bad_d] = bad
    out, _ = fp.flarepp_route(fp.ENCODE, q, k.to(td), v.to(td), want_lse=True)
    torch.cuda.synchronize()
    out = out[0, 0].cpu().numpy()
    assert np.isnan(out[:, bad_d]).all()
    keep = np.arange(D) != bad_d
    # bf16 weights of a uniform softmax over 128 tokens are all the same
    # number and cancel; what is left are fp32 sums of 128 terms
    np.testing.assert_allclose(out[:, keep], np.broadcast_to(want[keep], (M, D - 1)), rtol=0, atol=1e-5 * np.abs(want).max() + 1e-6)

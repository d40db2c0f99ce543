"""The decode of the forward that the backward runs, at C = 256, on both sides
of the line between the unfused and the fused kernel (tokens x routes 2^23, 2^22
and 2^20 at D = 16, 32 and 64): the training forward's output, the gradients of the pair against
the float64 oracle, and the stand-alone backward bitwise equal to the pair's.
Gate as for the other bf16 results.
"""

import pytest
import torch

from oracle import flarepp_oracle as orc
from paper_2608_11519_amd import flarepp as fp
from paper_2608_11519_amd import inputs as inp

from gpu_util import TOL, assert_close, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fp.load()
    yield


@pytest.mark.parametrize("N,H,M", [
    (16384, 4, 64), (16385, 4, 64), (16384, 8, 256), (16385, 8, 256), (32769, 16, 256),
])
def test_both_sides(N, H, M):
    C = 256
    w = inp.Workload("train-decode", 1, N, C, H, M, "bf16", "normal")
    assert fp.flarepp_mixer_path(fp.BF16, 1, N, C, H, M) == fp.PATH_FUSED
    print(f"[case] {inp.describe(w)}", flush=True)
    d = inp.make_inputs(w, 61, seed_scale=4.0)
    dO = inp.make_tensor((1, N, C), 62, "bf16")
    t = upload(d, w)
    args = (t["X"], t["Wk"], t["Wv"], t["Wkt"], t["Wvt"], t["Wo"], t["seeds"])
    dOt = torch.from_numpy(dO).to("cuda", t["X"].dtype)
    ws = torch.empty(fp.flarepp_mixer_backward_workspace_bytes(fp.BF16, 1, N, C, H, M), dtype=torch.uint8, device="cuda")
    O = fp.flarepp_mixer_forward_train(*args, H=H, ws=ws)
    a = fp.flarepp_mixer_backward_from_saved(*args, dOt, H=H, ws=ws)
    b = fp.flarepp_mixer_backward(*args, dOt, H=H)
    torch.cuda.synchronize()
    host = (d["X"], d["Wk"], d["Wv"], d["Wkt"], d["Wvt"], d["Wo"], d["seeds"])
    assert_close("O", O.float().cpu().numpy(), orc.mixer_forward(*host, H)["O"], TOL["bf16"], inp.describe(w))
    ref = orc.mixer_backward(*host, H, dO)
    for k, v in a.items():
        assert torch.equal(v, b[k]), k
        assert_close(k, v.float().cpu().numpy(), ref[k], TOL["bf16"], inp.describe(w))

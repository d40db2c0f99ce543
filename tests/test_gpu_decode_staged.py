"""GPU parity of the staged decode (C = 256) in its four- and eight-wave forms:
route counts on both sides of the line between them (224 / 256 at D = 16, 256 /
288 at D = 32, 96 / 128 at D = 64), token counts around a wave's and a
workgroup's tiles, forward and the statistics that the backward reads, against
the float64 oracle.  Gate as for the other bf16 results.
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


@pytest.mark.parametrize("B,N,H,M", [
    (1, 31, 8, 7), (2, 128, 8, 64), (1, 129, 8, 255), (2, 257, 8, 256), (1, 300, 8, 257),
    (1, 127, 16, 224), (1, 161, 16, 225), (1, 95, 4, 96), (2, 97, 4, 97),
])
def test_forms(B, N, H, M):
    C = 256
    w = inp.Workload("staged", B, N, C, H, M, "bf16", "normal")
    print(f"[case] {inp.describe(w)}", flush=True)
    d = inp.make_inputs(w, 31, seed_scale=4.0)
    dO = inp.make_tensor((B, N, C), 32, "bf16")
    t = upload(d, w)
    args = (t["X"], t["Wk"], t["Wv"], t["Wkt"], t["Wvt"], t["Wo"], t["seeds"])
    ref = orc.mixer_forward(d["X"], d["Wk"], d["Wv"], d["Wkt"], d["Wvt"], d["Wo"], d["seeds"], H)["O"]
    O = fp.flarepp_mixer_forward(*args, H=H)
    g = fp.flarepp_mixer_backward(*args, torch.from_numpy(dO).to("cuda", t["X"].dtype), H=H)
    torch.cuda.synchronize()
    assert_close("O", O.float().cpu().numpy(), ref, TOL["bf16"], inp.describe(w))
    rg = orc.mixer_backward(d["X"], d["Wk"], d["Wv"], d["Wkt"], d["Wvt"], d["Wo"], d["seeds"], H, dO)
    for k, v in g.items():
        assert_close(k, v.float().cpu().numpy(), rg[k], TOL["bf16"], inp.describe(w))

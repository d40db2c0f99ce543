"""GPU parity of the bf16 SDPA backward with the routes in registers (D = 16
and 32) at the edges of its work split, against the float64 oracle: one to
eight route groups, route counts around a block (32), a wave's blocks and a
workgroup's routes (1024 at D = 16, 512 at D = 32: a second launch adds to the
first), position counts around a tile and a step, more (batch, head) pairs
than compute units, widths without a fused forward.  Gate as for the other
bf16 gradients: 2e-2 of the reference's max |.|.
"""

import numpy as np
import pytest
import torch

from oracle import flarepp_oracle as orc
from paper_2608_11519_amd import flarepp as fp
from paper_2608_11519_amd import inputs as inp

from gpu_util import TOL, assert_close, upload

pytestmark = pytest.mark.gpu

GRADS = ("dX", "dWk", "dWv", "dWkt", "dWvt", "dWo", "dseeds", "dZ", "dQ")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fp.load()
    yield


def _grads(w, d, dO):
    t = upload(d, w)
    g = fp.flarepp_mixer_backward_debug(t["X"], t["Wk"], t["Wv"], t["Wkt"], t["Wvt"], t["Wo"], t["seeds"],
                                        torch.from_numpy(dO).to("cuda", t["X"].dtype), H=w.H)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in g.items()}


@pytest.mark.parametrize("B,N,C,H,M", [
    (1, 5, 64, 4, 3), (2, 31, 64, 4, 32), (1, 513, 64, 4, 33), (2, 512, 64, 4, 64), (1, 300, 64, 4, 65),
    (1, 4099, 128, 8, 128), (1, 777, 64, 4, 129), (1, 1000, 64, 4, 300), (1, 333, 64, 4, 1030),
    (20, 100, 128, 8, 64), (3, 2049, 32, 2, 16),
    (1, 33, 64, 2, 20), (2, 257, 64, 2, 64), (1, 1500, 128, 4, 100), (1, 700, 256, 8, 200), (1, 90, 64, 2, 530),
    (2, 450, 96, 6, 70), (1, 450, 96, 3, 140),
])
def test_route_and_position_edges(B, N, C, H, M):
    w = inp.Workload("bwd-edge", B, N, C, H, M, "bf16", "normal")
    print(f"[case] {inp.describe(w)}", flush=True)
    d = inp.make_inputs(w, 21, seed_scale=4.0)
    dO = inp.make_tensor((B, N, C), 22, "bf16")
    got = _grads(w, d, dO)
    ref = orc.mixer_backward(d["X"], d["Wk"], d["Wv"], d["Wkt"], d["Wvt"], d["Wo"], d["seeds"], H, dO)
    for k in GRADS:
        assert_close(k, got[k], ref[k], TOL["bf16"], inp.describe(w))


@pytest.mark.parametrize("sign", [-1.0, 1.0])
@pytest.mark.parametrize("C,H", [(64, 4), (64, 2)])
def test_large_scores_of_one_sign(C, H, sign):
    # Every score of the query synthesis is near +-256 (log2 units beyond the
    # fp32 exponent range), with position and route tails: the padded
    # positions and routes must not turn into inf * 0.  K~ = 16 X with X near
    # 1 and seeds 16 / sqrt(D), so a score is 16 * 16 * D / sqrt(D) / sqrt(D).
    # bf16 knows such scores to about 1 only, so the values are held to
    # finiteness.
    D = C // H
    w = inp.Workload("bwd-large", 1, 75, C, H, 40, "bf16", "normal")
    d = inp.make_inputs(w, 23)
    rng = np.random.default_rng(24)
    d["X"] = inp.round_to_bf16((1.0 + 2.0 ** -6 * rng.integers(-2, 3, d["X"].shape)).astype(np.float32))
    d["Wkt"] = inp.round_to_bf16(16.0 * np.eye(C, dtype=np.float32))
    d["seeds"] = np.full_like(d["seeds"], sign * D ** 0.5 / D * 16.0)
    got = _grads(w, d, inp.make_tensor((1, 75, C), 25, "bf16"))
    for k in GRADS:
        assert np.isfinite(got[k]).all(), k


@pytest.mark.parametrize("B,N,C,H", [(1, 1, 32, 2), (1, 70, 64, 4), (2, 1061, 128, 8), (1, 130, 512, 16), (1, 37, 1024, 16)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_block_layer_norm_gradients(B, N, C, H, dtype):
    # 4 to 64 lanes per token (C = 1024: two runs per lane), token counts
    # around a workgroup's chunk (1061 x 2 tokens: two per chunk, a short last
    # one)
    w = inp.Workload("ln-edge", B, N, C, H, 16, dtype, "normal")
    d = inp.make_inputs(w, 31)
    t = upload(d, w)
    gamma = inp.make_tensor((C,), 32, dtype) * 0.25 + 1
    gamma = inp.round_to_bf16(gamma) if dtype == "bf16" else gamma.astype(np.float32)
    beta = inp.make_tensor((C,), 33, dtype)
    dO = inp.make_tensor((B, N, C), 34, dtype)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", t["X"].dtype)  # noqa: E731
    g = fp.flarepp_block_backward(t["X"], up(gamma), up(beta), t["Wk"], t["Wv"], t["Wkt"], t["Wvt"], t["Wo"],
                                  t["seeds"], up(dO), H=H, eps=1e-5)
    torch.cuda.synchronize()
    ref = orc.block_backward(d["X"], gamma, beta, 1e-5, d["Wk"], d["Wv"], d["Wkt"], d["Wvt"], d["Wo"], d["seeds"], H, dO)
    for k in ("dX", "dgamma", "dbeta"):
        assert_close(k, g[k].cpu().numpy(), ref[k], TOL[dtype], inp.describe(w))

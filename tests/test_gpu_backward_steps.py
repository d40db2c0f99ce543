"""The loops of the bf16 backward past their first pass: several steps, tiles or
ring turns per workgroup with a ragged last one, against the float64 oracle.
Every case asserts from the split rules that it has them.  Gate as for the
other bf16 gradients: 2e-2 of the reference's max |.|, and for dseeds the bound
below where that is larger.
"""

import numpy as np
import pytest
import torch

import split_rules as sr
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


def _seed_bound(d, H):
    """Largest relative error of a softmax weight of the query synthesis.  Its
    score is a sum of D products of operands rounded to bf16 (2^-9 each), so it
    is off by at most 2^-8 sum_d |q_d k_d| / sqrt(D), and exp turns that into a
    relative error.  With hundreds of sharp seeds over a few hundred tokens a
    route's gradient can hang on one such weight, which is then the largest
    error of dseeds (2.5e-2 here with M = 700, the same to three digits in two
    unlike implementations; the 2-norm error is 6e-3)."""
    K = np.abs(orc.project(d["X"], d["Wkt"], H)).astype(np.float32)  # [B, H, N, D]
    q = np.abs(np.asarray(d["seeds"], dtype=np.float32))              # [H, M, D]
    return 2.0 ** -8 * max(float((K[:, h] @ q[h].T).max()) for h in range(H)) / q.shape[-1] ** 0.5


def _check(B, N, C, H, M, train=False):
    w = inp.Workload("bwd-steps", B, N, C, H, M, "bf16", "normal")
    print(f"[case] {inp.describe(w)}", flush=True)
    d = inp.make_inputs(w, 71, seed_scale=4.0)
    dO = inp.make_tensor((B, N, C), 72, "bf16")
    t = upload(d, w)
    args = (t["X"], t["Wk"], t["Wv"], t["Wkt"], t["Wvt"], t["Wo"], t["seeds"])
    dOt = torch.from_numpy(dO).to("cuda", t["X"].dtype)
    host = (d["X"], d["Wk"], d["Wv"], d["Wkt"], d["Wvt"], d["Wo"], d["seeds"])
    if train:
        ws = torch.empty(fp.flarepp_mixer_backward_workspace_bytes(fp.BF16, B, N, C, H, M), dtype=torch.uint8,
                         device="cuda")
        O = fp.flarepp_mixer_forward_train(*args, H=H, ws=ws)
        g = fp.flarepp_mixer_backward_from_saved(*args, dOt, H=H, ws=ws)
        torch.cuda.synchronize()
        assert_close("O", O.float().cpu().numpy(), orc.mixer_forward(*host, H)["O"], TOL["bf16"])
    else:
        g = fp.flarepp_mixer_backward_debug(*args, dOt, H=H)
        torch.cuda.synchronize()
    ref = orc.mixer_backward(*host, H, dO)
    for k, v in g.items():
        got = v.float().cpu().numpy()
        tol = max(TOL["bf16"], _seed_bound(d, H)) if k == "dseeds" else TOL["bf16"]
        assert_close(k, got, ref[k], tol, inp.describe(w))
        if k == "dX":  # the last tokens of the last batch entry, at the same gate
            assert np.abs(got[-1, -40:] - ref[k][-1, -40:]).max() <= TOL["bf16"] * np.abs(ref[k]).max()


# 256 (batch, head) pairs: one workgroup each.  rb route blocks per wave, rw
# route groups, launches over the routes.
@pytest.mark.parametrize("B,N,H,M,rb,rw,launches", [
    (64, 1613, 4, 20, 1, 1, 1), (64, 1100, 4, 50, 2, 1, 1), (64, 1100, 4, 128, 4, 1, 1), (64, 600, 4, 200, 4, 2, 1),
    (64, 300, 4, 500, 4, 4, 1), (64, 200, 4, 700, 4, 8, 1), (64, 150, 4, 1030, 4, 8, 2),
    (128, 809, 2, 20, 1, 1, 1), (128, 600, 2, 64, 2, 1, 1), (128, 300, 2, 100, 2, 2, 1), (128, 150, 2, 200, 2, 4, 1),
    (128, 100, 2, 400, 2, 8, 1), (128, 75, 2, 530, 2, 8, 2),
])
def test_sdpa_backward_several_steps(B, N, H, M, rb, rw, launches):
    C = 64
    s = sr.rs_split(B, H, N, C // H, M)
    assert (s["rb"], s["rw"], s["R"]) == (rb, rw, 1) and s["steps"] >= 3 and N % s["positions"]
    assert -(-((M + 31) // 32) // s["nbw"]) == launches
    _check(B, N, C, H, M)


# the token products: T tokens, T / 32 tiles over the 2,048 waves of k_rows_sum
# and of one weight's projection (C <= 128), T / 64 over the 256 workgroups of
# k_rows_sum_stream (C = 256), k_wgrad's rings of 12, 8 and 4 steps of 32 tokens
@pytest.mark.parametrize("N,C,H,M,ring", [(150001, 64, 4, 8, 12), (140003, 128, 8, 8, 8), (140001, 256, 16, 8, 4),
                                           (140001, 256, 8, 40, 4)])
def test_token_products_several_tiles(N, C, H, M, ring):
    assert N > 2 * 2048 * 32 and N % 64
    chunks, chunk = sr.wgrad_chunks(N)
    assert chunk // 32 > 3 * ring and (N - (chunks - 1) * chunk) % 32
    _check(1, N, C, H, M, train=True)


def test_projection_several_tiles_wide():
    # C = 256, one weight per workgroup: 4,137 tiles of 32 tokens over the 512
    # waves of each of four weights, and over the 2,048 waves of one
    w = inp.Workload("proj-wide", 3, 44101, 256, 8, 8, "bf16", "normal")
    d = inp.make_inputs(w, 73)
    t = upload(d, w)
    outs = fp.flarepp_project(t["X"], t["Wk"], t["Wv"], t["Wkt"], t["Wvt"], H=w.H)
    torch.cuda.synchronize()
    for name, W, got in zip(("K", "V", "Kt", "Vt"), ("Wk", "Wv", "Wkt", "Wvt"), outs):
        assert_close(name, got.float().cpu().numpy(), orc.project(d["X"], d[W], w.H), TOL["bf16"] / 2, "project-wide")
    _, _, Kt1, _ = fp.flarepp_project(t["X"], Wkt=t["Wkt"], H=w.H)
    torch.cuda.synchronize()
    assert torch.equal(Kt1, outs[2])


@pytest.mark.parametrize("N", [33, 128, 129, 8192, 8193])
def test_projection_forms_wide(N):
    # C = 256, four weights: the persistent form up to 4 tiles of 32 tokens and
    # from 1,025 tiles x weights on, the general one between
    w = inp.Workload("proj-forms", 1, N, 256, 16, 8, "bf16", "normal")
    d = inp.make_inputs(w, 74)
    t = upload(d, w)
    outs = fp.flarepp_project(t["X"], t["Wk"], t["Wv"], t["Wkt"], t["Wvt"], H=w.H)
    torch.cuda.synchronize()
    for name, W, got in zip(("K", "V", "Kt", "Vt"), ("Wk", "Wv", "Wkt", "Wvt"), outs):
        assert_close(name, got.float().cpu().numpy(), orc.project(d["X"], d[W], w.H), TOL["bf16"] / 2, f"project-{N}")

"""The merge of an encode's split-key partials: chunk counts around the edges
of its batches and of its two forms (and empty chunks) and the norm bounds that
it writes for the decode, against the float64 oracle; values that are not
finite, against what the softmax defines for them (a zero weight times an
infinity or a NaN is a NaN).
"""

import numpy as np
import pytest
import torch

from oracle import flarepp_oracle as orc
from paper_2608_11519_amd import flarepp as fp
from paper_2608_11519_amd import inputs as inp

from gpu_util import TOL, assert_close, run_mixer

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


# four, two and one slices of up to 8 chunks at D = 16, 32 and 64, then batches
# of 64 chunks (the last one of up to 32)
@pytest.mark.parametrize("D,chunks", [
    (16, 1), (16, 4), (16, 5), (16, 9), (16, 17), (16, 32), (16, 33), (16, 64), (16, 65), (16, 97), (16, 200),
    (32, 2), (32, 3), (32, 5), (32, 9), (32, 16), (32, 17), (32, 63), (32, 96), (32, 130),
    (64, 1), (64, 2), (64, 3), (64, 5), (64, 8), (64, 9), (64, 33), (64, 64), (64, 128), (64, 161),
])
def test_chunk_counts(monkeypatch, D, chunks):
    monkeypatch.setenv("FLAREPP_FORCE_CHUNKS", str(chunks))
    B, H, M = 2, 1, 37
    N = 32 * chunks - 13 if chunks % 2 else 20 * chunks + 7  # even counts: empty chunks at the end
    q = inp.make_tensor((B, H, M, D), 51, "f32", scale=2.0)
    k = inp.make_tensor((B, H, N, D), 52, "f32")
    v = inp.make_tensor((B, H, N, D), 53, "f32")
    out, lse = fp.flarepp_route(fp.ENCODE, *(torch.from_numpy(x).cuda() for x in (q, k, v)), want_lse=True)
    torch.cuda.synchronize()
    ref, L = orc.sdpa(q, k, v)
    assert_close("out", out.cpu().numpy(), ref, TOL["f32"], f"D{D} R{chunks}")
    np.testing.assert_allclose(lse.cpu().numpy(), L, rtol=0, atol=1e-4)


# more rows than two workgroups per CU hold: several batches of 8 per slice
@pytest.mark.parametrize("D,B,chunks", [(16, 150, 33), (16, 150, 70), (32, 80, 17), (32, 80, 35), (64, 40, 9), (64, 40, 21)])
def test_chunk_counts_of_many_rows(monkeypatch, D, B, chunks):
    monkeypatch.setenv("FLAREPP_FORCE_CHUNKS", str(chunks))
    H, M, N = 1, 90, 32 * chunks - 13
    assert B * H * 96 * D > 512 * 256
    q = inp.make_tensor((B, H, M, D), 56, "f32", scale=2.0)
    k = inp.make_tensor((B, H, N, D), 57, "f32")
    v = inp.make_tensor((B, H, N, D), 58, "f32")
    out, lse = fp.flarepp_route(fp.ENCODE, *(torch.from_numpy(x).cuda() for x in (q, k, v)), want_lse=True)
    torch.cuda.synchronize()
    ref, L = orc.sdpa(q, k, v)
    assert_close("out", out.cpu().numpy(), ref, TOL["f32"], f"D{D} R{chunks}")
    np.testing.assert_allclose(lse.cpu().numpy(), L, rtol=0, atol=1e-4)


@pytest.mark.parametrize("chunks", [1, 200])
@pytest.mark.parametrize("row", [0, 1, 2, 3, 30])
@pytest.mark.parametrize("D", [16, 32, 64])
def test_norm_bound_of_every_row(monkeypatch, D, row, chunks):
    # Identity weights.  Token 7 is 30 e0 and one seed finds it, so that
    # route's query and latent are 30 e0 and token 7's score with it is
    # 900 / sqrt(D): beyond the fp32 exponent range without a shift, which the
    # decode leaves out unless the bound of the route's group says so.
    C, M = 64, 32
    N = 32 * chunks if chunks > 1 else 64
    monkeypatch.setenv("FLAREPP_FORCE_CHUNKS", str(chunks))
    w = inp.Workload("bound", 1, N, C, C // D, M, "bf16", "normal")
    eye = np.eye(C, dtype=np.float32)
    X = inp.round_to_bf16(0.1 * inp.make_tensor((1, N, C), 54, "f32"))
    seeds = inp.round_to_bf16(0.1 * inp.make_tensor((C // D, M, D), 55, "f32"))
    X[0, 7] = 0
    for h in range(C // D):
        X[0, 7, h * D] = 30
        seeds[h, row] = 0
        seeds[h, row, 0] = 40
    d = dict(X=X, Wk=eye, Wv=eye, Wkt=eye, Wvt=eye, Wo=eye, seeds=seeds)
    assert fp.flarepp_mixer_path(fp.BF16, 1, N, C, C // D, M) == fp.PATH_FUSED
    got = run_mixer(d, w)
    ref = orc.mixer_forward(X, eye, eye, eye, eye, eye, seeds, C // D)
    for k in ("Q", "Z", "Y", "O"):
        assert_close(k, got[k], ref[k], TOL["bf16"], f"D{D} row{row}")

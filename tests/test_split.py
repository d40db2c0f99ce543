"""Work splits of the backward on the host: every position, route and token is
covered once, and no chunk count takes longer than the plain rules would."""

import pytest

import split_rules as sr


def _cdiv(a, b):
    return -(-a // b)


@pytest.mark.parametrize("D,elem_bytes", [(16, 4), (32, 4), (64, 4), (64, 2)])
@pytest.mark.parametrize("dec", [False, True])
def test_bwd_split_rounds(D, elem_bytes, dec):
    # two plain rules: chunks that fit one round of 256 workgroups, and about
    # 512 workgroups in all; the first leaves CUs idle from 129 pairs on, the
    # second runs a nearly empty last round
    for Mp in (32, 128, 320):
        for tiles in (1, 7, 63, 625, 2000):
            for BH in list(range(1, 400)) + [512, 513, 600, 768, 1000, 4096]:
                s = sr.bwd_split(BH, 32 * tiles - 5, D, Mp, dec, elem_bytes)
                W, R = s["waves"], s["R"]
                assert W in (1, 2, 4) and 1 <= s["nsb"] <= Mp // 32
                assert (R - 1) * s["tpw"] * W < tiles <= R * s["tpw"] * W
                assert R <= max(1, _cdiv(512, BH))  # no more partials than the second rule's
                most = _cdiv(tiles, W)
                for plain in (max(1, min(256 // BH, most)), min(_cdiv(512, BH), most)):
                    assert sr.rounds_time(BH, tiles, W, R) <= sr.rounds_time(BH, tiles, W, plain), (BH, tiles, R, plain)


@pytest.mark.parametrize("D", [16, 32])
def test_rs_split_covers_the_positions(D):
    for M in (8, 33, 64, 100, 128, 200, 512, 1030):
        for N in (5, 513, 4099, 50000):
            for B, H in [(1, 1), (1, 4), (2, 8), (12, 8), (20, 8), (32, 8), (130, 4)]:
                s = sr.rs_split(B, H, N, D, M)
                span = s["positions"] * s["steps"]
                assert (s["R"] - 1) * span < N <= s["R"] * span
                assert s["nbw"] == s["rb"] * s["rw"] and (s["nbw"] * 32 >= M or s["rw"] == 8)


def test_wgrad_chunks_cover_the_tokens():
    for T in (1, 127, 128, 129, 5000, 100000, 1 << 20):
        for nprob in (5, 7):
            n, c = sr.wgrad_chunks(T, nprob)
            assert c % 32 == 0 and (n - 1) * c < T <= n * c and n * nprob <= 256

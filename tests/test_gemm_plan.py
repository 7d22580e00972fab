"""Which kernel a product takes (host arithmetic, no GPU): the choice stays inside the room the workspace query names, never splits
without it, and follows the number of compute units."""
import random

import pytest

from paper_2505_20524_amd import fog


def shapes(n, seed):
    rng = random.Random(seed)
    for _ in range(n):
        M, N, K = (round(2 ** rng.uniform(4, 14)) for _ in range(3))
        yield rng.choice([fog.NT, fog.NN, fog.TN]), M, N, K


def test_partial_tiles_fit_the_room():
    split = 0
    for layout, M, N, K in shapes(4000, 1):
        tm, tn, _, splits, k_chunk = fog.probe_gemm_plan(layout, M, N, K, True, 0)
        room = fog.fp8_gemm_workspace(layout, M, N, K)
        assert splits == -(-K // k_chunk) and (splits == 1 or (k_chunk >= 512 and k_chunk % 128 == 0))
        if splits > 1:
            split += 1
            assert splits * -(-M // tm) * -(-N // tn) * tm * tn * 4 <= room
        assert fog.probe_gemm_plan(layout, M, N, K, False, 0)[3] == 1
    assert split > 100


def test_every_kernel_is_chosen_somewhere():
    seen = {(layout, ws): set() for layout in (fog.NT, fog.NN, fog.TN) for ws in (False, True)}
    for layout, M, N, K in shapes(20000, 2):
        for ws in (False, True):
            tm, tn, per_cu, splits, _ = fog.probe_gemm_plan(layout, M, N, K, ws, 256)
            if ws == (splits > 1):
                seen[layout, ws].add((tm, tn, per_cu))
    for layout in (fog.NT, fog.NN, fog.TN):
        assert seen[layout, False] == {(256, 256, 1), (256, 128, 1), (128, 128, 1), (128, 128, 2), (64, 64, 2)}
        assert seen[layout, True] == {(256, 256, 1), (256, 128, 1), (128, 128, 1), (64, 64, 2)}


def test_the_choice_follows_the_compute_units():
    """32 tiles of 256 x 256 leave most of 256 compute units idle and fill a partition of 32."""
    assert fog.probe_gemm_plan(fog.NT, 2048, 1024, 4096, False, 256)[:2] != (256, 256)
    assert fog.probe_gemm_plan(fog.NT, 2048, 1024, 4096, False, 32)[:2] == (256, 256)


def test_plan_errors():
    for args in [(fog.NT, 0, 16, 16), (fog.NT, 16, -1, 16), (fog.NT, 16, 16, 2 ** 31), (7, 16, 16, 16)]:
        with pytest.raises(fog.FogError):
            fog.probe_gemm_plan(*args)

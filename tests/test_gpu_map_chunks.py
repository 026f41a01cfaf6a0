"""Task-map build at the edges of its launch shapes (one workgroup of as many wavefronts as rows or experts need; one
launch that counts all ids in every workgroup; two launches), with and without ids outside [0, E)."""
import numpy as np
import pytest
import torch

from paper_2501_16103_amd import binding as mb

pytestmark = pytest.mark.gpu

CHUNK = 1024
CASES = [(R, E) for R in (1, 64, 65, CHUNK, CHUNK + 1, 16 * CHUNK, 16 * CHUNK + 1, 70 * CHUNK + 5) for E in (1, 64, 65, 192, 1024)]


@pytest.mark.parametrize("order", [0, 1, 2], ids=["ascending", "spread", "interleave"])
@pytest.mark.parametrize("bad", [False, True], ids=["valid", "bad_ids"])
def test_map_build_chunk_edges(order, bad):
    dev = torch.device("cuda:0")
    for R, E in CASES:
        rng = np.random.default_rng(R * 1031 + E)
        ids = np.minimum(rng.geometric(4.0 / (E + 3), R) - 1, E - 1).astype(np.int32)     # skewed, with empty experts
        nbad = 0
        if bad:
            where = np.unique(np.concatenate([rng.integers(0, R, 1 + R // 50), [0, R - 1]]))
            ids[where] = rng.choice([-1, E, E + 1, 2 ** 31 - 1, -2 ** 31], len(where))
            nbad = len(where)
        tmap = mb.alloc_task_map(R, 1, E, 64, 128, 384, dev)
        tmap.fill_(0x5A5A5A5A)
        mb.moe_build_task_map_ordered(torch.from_numpy(ids).to(dev), R, 1, E, 64, 128, 384, order, tmap)
        got, o, hdr = tmap.cpu().numpy(), mb.moe_map_offsets(E), mb.HDR
        ok = (ids >= 0) & (ids < E)
        counts = np.bincount(ids[ok], minlength=E)
        tiles = (counts + 63) // 64 * 3
        M = int((counts > 0).sum())
        assert got[hdr["STATUS"]] == nbad and got[hdr["M"]] == M and got[hdr["R"]] == R
        assert got[hdr["TOTAL_TILES"]] == (0 if nbad else tiles.sum())
        np.testing.assert_array_equal(got[o["counts"]: o["counts"] + E], counts, err_msg=f"R={R} E={E}")
        offsets = np.concatenate([[0], np.cumsum(counts)])
        np.testing.assert_array_equal(got[o["offsets"]: o["offsets"] + E + 1], offsets, err_msg=f"R={R} E={E}")
        rows = np.flatnonzero(ok)[np.argsort(ids[ok], kind="stable")]
        np.testing.assert_array_equal(got[o["sorted_rows"]: o["sorted_rows"] + len(rows)], rows, err_msg=f"R={R} E={E}")
        sigma = got[o["sigma"]: o["sigma"] + M]
        np.testing.assert_array_equal(np.sort(sigma), np.flatnonzero(counts))
        if order == 0:
            np.testing.assert_array_equal(sigma, np.flatnonzero(counts))
        np.testing.assert_array_equal(got[o["tile_prefix"]: o["tile_prefix"] + M], np.cumsum(tiles[sigma]))
        rec = got[o["task_records"]: o["task_records"] + 4 * ((E + 63) // 64 * 64)].reshape(-1, 4)
        np.testing.assert_array_equal(rec[:M], np.stack([np.cumsum(tiles[sigma]), sigma, counts[sigma], offsets[sigma]], axis=1))
        np.testing.assert_array_equal(rec[M:], np.tile([2 ** 31 - 1, -1, 0, 0], (len(rec) - M, 1)))
        if R > CHUNK:   # scratch: one histogram per chunk (experts, bad ids, spare columns), the same from one launch or two
            E64, at = (E + 63) // 64 * 64, o["sorted_rows"] + (R + 63) // 64 * 64
            for c in range((R + CHUNK - 1) // CHUNK):
                part, line = ids[c * CHUNK: (c + 1) * CHUNK], got[at + c * (E64 + 64): at + (c + 1) * (E64 + 64)]
                good = (part >= 0) & (part < E)
                want = np.concatenate([np.bincount(part[good], minlength=E64), [(~good).sum()], np.zeros(63, int)])
                np.testing.assert_array_equal(line, want, err_msg=f"R={R} E={E} chunk {c}")
        assert np.all(got[o["sigma"] + M: o["tile_prefix"]] == -1) and np.all(got[o["tile_prefix"] + M: o["task_records"]] == 2 ** 31 - 1)


@pytest.mark.parametrize("order", [0, 1, 2], ids=["ascending", "spread", "interleave"])
def test_map_pair_equals_two_builds(order):
    """One build of both maps of a layer: the bytes of the two separate builds, bad ids included."""
    dev = torch.device("cuda:0")
    g1, g2 = mb.Tiling(64, 128, order, 16, 40), mb.Tiling(256, 256, 2 - order, 0, 0, 32)
    for T, k, E, bad in ((0, 2, 8, 0), (1, 6, 64, 0), (170, 6, 100, 3), (171, 6, 64, 0), (2500, 4, 1000, 0), (8192, 3, 8, 7)):
        rng = np.random.default_rng(T + E)
        ids = rng.integers(0, E, (T, k)).astype(np.int32)
        ids.reshape(-1)[:bad] = -1
        ids = torch.from_numpy(ids).to(dev)
        R, N1, N2 = T * k, 896, 512
        maps = [mb.alloc_task_map(max(T, 1), k, E, 64, 128, N1, dev).fill_(7) for _ in range(2)]
        maps += [mb.alloc_task_map(max(R, 1), 1, E, 256, 256, N2, dev).fill_(7) for _ in range(2)]
        mb.moe_build_task_map_ex(ids, T, k, E, N1, g1, maps[0])
        mb.moe_build_task_map_ex(ids.reshape(R, 1), R, 1, E, N2, g2, maps[2])
        mb.moe_build_task_map_pair(ids, T, k, E, N1, g1, maps[1], N2, g2, maps[3])
        used = mb.moe_map_offsets(E)["sorted_rows"] + R - bad
        for a, b in ((0, 1), (2, 3)):
            assert torch.equal(maps[a][:used], maps[b][:used]), (T, k, E, a)
            if bad == 0:
                assert torch.equal(maps[a], maps[b]), (T, k, E, a, "scratch")
    assert mb.moe_build_task_map_pair(ids, T, k, E, N1, g1, maps[1], N2, g2, maps[1], check=False) == mb.MOE_ERR_INVALID_ARG

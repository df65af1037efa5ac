"""Host mirror of the partitions by pairs (no GPU): every pair's parts cover it,
fit the work groups and keep to the largest part; short pairs stay whole."""
import numpy as np
import pytest

import paper_2506_03296_amd as A


@pytest.mark.parametrize("seed", range(8))
def test_parts_cover_every_pair_and_fit_the_work_groups(seed):
    rng = np.random.default_rng(seed)
    applied = whole = 0
    for _ in range(300):
        B = int(np.exp(rng.uniform(0, np.log(600))))
        hi = int(np.exp(rng.uniform(np.log(2), np.log(20000))))
        lens = rng.integers(-1, hi, size=B)
        Hkv = int(rng.choice([1, 2, 8, 16, 32, 80]))
        G = int(rng.choice([1, 2, 4, 8]))
        cus, launched = [(256, 512), (256, 256), (32, 64), (0, 512)][int(rng.integers(0, 4))]
        p = A.plan_pairs_host(lens, G * Hkv, Hkv, launched, cus)
        blocks = np.where(lens > 0, -(-lens // 16), 0)
        pairs, units, longest = int((blocks > 0).sum()) * Hkv, int(blocks.sum()) * Hkv, int(blocks.max())
        groups = min(cus, launched) if pairs <= cus else launched
        fits = cus > 0 and B <= 256 and 0 < pairs <= groups and (longest <= 32 or units <= 24 * (groups - pairs))
        short = (cus > 0 and not fits and B <= 512 and pairs > launched and longest <= 32
                 and (30 + 12 * longest) * launched <= 70 * pairs + 5 * units
                 and (pairs <= 4 * launched or pairs > 8 * launched or longest <= 24 or units <= 12 * pairs
                      or 8 * units > 7 * longest * pairs))
        assert (p["active"] > 0) == (fits or short)
        if short:
            whole += 1
            assert p["active"] == launched
            assert np.array_equal(p["parts"], blocks > 0) and np.array_equal(p["part_units"], blocks)
            continue
        if not fits:
            assert not p["parts"].any()
            continue
        applied += 1
        parts, T = p["parts"].astype(np.int64), p["part_units"].astype(np.int64)
        assert p["active"] == int(parts.sum()) * Hkv <= groups
        assert np.all((parts == 0) == (blocks == 0))
        used = blocks > 0
        assert np.all((parts[used] - 1) * T[used] < blocks[used])      # no empty part
        assert np.all(parts[used] * T[used] >= blocks[used])           # nothing left over
        assert np.all(parts[blocks <= 16] <= 1)
    assert applied > 20 and whole > 5


# Batches measured on the line and by waves (us, line / waves, on 256 CUs and 512
# work groups): the partition that was faster.  (lens, Hkv, by waves)
MEASURED = [
    ([20 + 4 * (i % 11) for i in range(256)], 8, True),            # 21.2 / 11.5
    ([16 + i % 33 for i in range(300)], 8, True),                  # 22.6 / 13.2
    ([200 + 4 * (i % 15) for i in range(256)], 8, True),           # 46.3 / 38.7
    ([200 + 4 * (i % 15) for i in range(80)], 8, False),           # 20.9 / 27.2
    ([277 + 59 * (i % 2) for i in range(286)], 8, True),           # 72.6 / 65.1
    ([16 + 31 * i % 497 for i in range(144)], 16, False),          # 62.7 / 66.1
    ([16 + 31 * i % 497 for i in range(188)], 16, False),          # 74.6 / 78.4
    ([310 + 168 * (i % 2) for i in range(82)], 32, False),         # 89.4 / 97.5
    ([34 + 432 * (i % 2) for i in range(262)], 8, False),          # 57.0 / 60.4
    ([128 + 384 * (i % 16 == 0) for i in range(144)], 16, True),   # 46.0 / 37.3
    ([512] * 257, 16, True),                                       # 175.1 / 170.4
    ([1] * 176 + [512] * 12, 16, True),                            # 34.3 / 24.4
    ([16 + 31 * i % 497 for i in range(388)], 16, True),           # 162.4 / 153.8
]


@pytest.mark.parametrize("lens,Hkv,waves", MEASURED)
def test_measured_batches_take_the_faster_partition(lens, Hkv, waves):
    p = A.plan_pairs_host(lens, 4 * Hkv, Hkv, 512, 256)
    assert len(lens) * Hkv > 512 and p["active"] == (512 if waves else 0)


# The same for the line and the pair cut: (lens, Hq, Hkv, parts)
MEASURED_CUTS = [
    ([300], 32, 8, True),                                          # 10.8 / 7.2
    ([2100], 32, 8, True),                                         # 12.6 / 10.1
    ([20 + 3 * (i % 61) for i in range(64)], 8, 8, True),          # 13.5 / 10.8
    ([676 - 560 * (i % 2) for i in range(135)], 2, 2, False),      # 18.8 / 21.0
    ([383 + 130 * (i % 4 == 0) for i in range(17)], 16, 16, False),   # 18.8 / 21.0
    ([1267] * 8, 8, 8, False),                                     # 12.1 / 13.1
]


@pytest.mark.parametrize("lens,Hq,Hkv,parts", MEASURED_CUTS)
def test_measured_batches_are_cut_where_parts_are_faster(lens, Hq, Hkv, parts):
    p = A.plan_pairs_host(lens, Hq, Hkv, 512, 256)
    assert len(lens) * Hkv <= 512 and (p["active"] > 0) == parts


def test_bad_arguments_are_refused():
    for args in (([5], 8, 0, 512, 256), ([5], 7, 2, 512, 256), ([5], 8, 2, 0, 256), ([5], 8, 2, 512, -1)):
        with pytest.raises(A.ApexError):
            A.plan_pairs_host(*args)
    with pytest.raises(A.ApexError):
        A.plan_pairs_host([5], 8, 2, 512, 256, block_size=32)
    assert A.plan_pairs_host([], 8, 2, 512, 256)["active"] == 0

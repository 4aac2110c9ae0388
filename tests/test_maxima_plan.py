"""When a small batch goes by group maxima, and what the plan must hold for the kernels (no device needed)."""
import pytest

from paper_2110_08919_amd import lpq


@pytest.mark.parametrize("d,bits,packed,n,nq,k,taken", [
    (128, 8, False, 20_000, 256, 10, True), (128, 8, False, 1_000_000, 64, 128, True), (128, 8, False, 1_000_000, 64, 129, False),
    (128, 4, False, 100_000, 1, 10, True), (128, 3, False, 100_000, 1, 10, False), (63, 6, False, 100_000, 1, 10, True),
    (63, 5, False, 100_000, 1, 10, False), (64, 5, False, 100_000, 1, 10, True), (128, 4, True, 100_000, 64, 20, True),
    (128, 4, True, 3_000_000, 8, 10, True), (128, 4, True, 3_000_001, 8, 10, False),
    (4096, 8, False, 20_000, 4, 10, True), (4097, 8, False, 20_000, 4, 10, False), (400, 8, False, 20_000, 512, 1, True),
    (400, 8, False, 20_000, 513, 1, False), (64, 8, False, 4096, 2048, 5, True), (64, 8, False, 4096, 2049, 5, False),
    (128, 8, False, 1_000_000, 100, 10, True), (128, 8, False, 1_000_000, 640, 10, False),
    # groups in sixteens: below 65 536 rows an even number of stages, of two waves a multiple of four
    (128, 8, False, 128 * 78, 100, 10, True), (128, 8, False, 128 * 79, 100, 10, False), (200, 8, False, 64 * 160, 100, 10, True),
    (200, 8, False, 64 * 162, 100, 10, False),
    # streamed rows: few sets of groups for k, and so most rows scored again; few rows or few queries all the same
    (1913, 8, False, 12_902, 64, 50, False), (647, 8, False, 26_441, 84, 100, False), (653, 8, False, 14_474, 152, 50, False),
    (2777, 8, False, 5908, 4, 23, True), (3432, 8, False, 6551, 242, 10, True), (978, 8, False, 53_042, 64, 100, True),
])
def test_which_batches_take_group_maxima(d, bits, packed, n, nq, k, taken):
    assert (lpq.search_maxima_info(d, bits, packed, n, nq, k)[0] > 0) == taken


@pytest.mark.parametrize("key", [lpq.TUNE_PATH, lpq.TUNE_SPLITS, lpq.TUNE_SEED_ROWS, lpq.TUNE_WAVE_QUERIES, lpq.TUNE_REGION_CAP])
def test_a_tuned_search_does_not(key):
    lpq.set_tuning(key, {lpq.TUNE_PATH: 3, lpq.TUNE_WAVE_QUERIES: 64}.get(key, 512))
    try:
        assert not any(lpq.search_maxima_info(128, 8, False, 1_000_000, 16, 10))
    finally:
        lpq.set_tuning(key, 0)


@pytest.mark.parametrize("d", [24, 64, 100, 128, 192, 256, 300, 700, 1500, 4096])
def test_what_the_kernels_ask_for(d):
    taken = 0
    for packed in (False, True):
        if packed and d > 256:
            continue
        for n in (4096, 4223, 5003, 9999, 10_112, 20_577, 32_768, 65_535, 65_536, 131_135, 300_001, 1_000_000, 10_000_000):
            for nq in (1, 3, 16, 63, 64, 65, 128, 129, 200, 512, 513, 2048, 4096, 4097):
                for k in (1, 10, 33, 100, 128) if packed else (1, 10, 33, 100, 128, 129):
                    G, S, SEG, waves, stage, threads, helpers, most = lpq.search_maxima_info(d, 4 if packed else 8, packed, n, nq, k)
                    if not G:
                        continue
                    taken += 1
                    what = (d, packed, n, nq, k)
                    per_tile = min(nq, 64) if packed else nq
                    assert stage == 32 * waves and waves == (8 if d > 256 else 2 if not packed and d > 128 else 4), what
                    assert G == S * SEG * 2 * waves and G % 16 == 0 and G <= 16 * threads and threads in (256, 1024), what
                    assert 1 <= SEG <= n // stage // S and (S <= 512 if waves < 8 else S <= 256), what     # no segment without rows
                    assert k <= 128 and min(256, G // 4 if threads == 256 else G // 16) >= k, what        # sets for the bound
                    assert n - n // stage * stage <= 256 and d <= 4096 and per_tile <= 4096, what
                    assert 1 <= helpers <= most <= 16 and most * k <= 2048, what
                    info = lpq.search_plan_info(d, 4 if packed else 8, packed, n, nq, k)
                    assert info[24] + per_tile * G * 4 <= info[34] <= info[16], what                       # the maxima fit
    assert taken > 100


def test_arguments():
    L = lpq.lib()
    out = (lpq.C.c_int64 * 8)()
    assert L.lpq_search_maxima_info(128, 8, 0, 1000, 10, 10, out, 7) == lpq.EINVAL
    assert L.lpq_search_maxima_info(128, 8, 0, 1000, 10, 10, None, 8) == lpq.EINVAL
    assert L.lpq_search_maxima_info(128, 9, 0, 1000, 10, 10, out, 8) == lpq.EINVAL
    assert L.lpq_search_maxima_info(128, 8, 0, 1000, 10, 2000, out, 8) == lpq.ERANGE
    assert L.lpq_search_maxima_info(128, 8, 0, 1000, 10, 10, out, 8) == lpq.OK and not any(out)

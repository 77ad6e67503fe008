"""The route rules over the sizes they accept: what they return has to fit the kernels' own limits."""
import itertools

from tests import rules


def test_rules_stay_within_the_kernels_limits():
    L = rules.lib()
    dims = [64, 128, 192, 256, 320, 512, 576, 768, 1024, 1088, 2048, 4096, 8192]
    for dt, m, n, k in itertools.product((0, 1), (1, 2, 4, 5, 8, 12, 16, 17, 64, 65, 128, 300, 1000, 4096), dims + [1004, 18428, 32000], dims):
        ks = L.pick_ksplit(m, n, k, dt)
        assert 1 <= ks <= 16 and ks & (ks - 1) == 0
        if dt == 0:
            wm, sp = L.split_wm(m, n, k, 1, 4), L.split_ks(m, n, k, 1, 4)
            assert wm in (0, 2, 3) and (wm == 0 or k % (64 * sp) == 0)
            # the split of a product that writes partials is the one its launch asks for again
            assert wm == 0 or (ks == sp and L.split_wm(m, n, k, sp, sp) == wm)
        for kind in (0, 1, 2, 3):
            assert not L.skinny(dt, m, n, k, kind, 1) or (m <= 16 and k % (32 if dt else 16) == 0)
            assert not L.skinny(dt, m, n, k, kind, 2) or kind == 3
    for dt, rows, d in itertools.product((0, 1), range(1, 40), range(64, 2049, 64)):
        assert not L.few_rows(dt, rows, d) or (rows <= 16 and d <= 1024)
    for n in (4, 1000, 18428, 18432, 32000):
        assert L.cand_n(n) in (64, 128)


def test_bf16_products_get_a_tile_that_can_take_them():
    L = rules.lib()
    chunk = [128, 64, 64, 64, 64, 64, 64]
    seen = set()
    for kind, ragged in ((0, 0), (0, 1), (1, 0), (2, 0), (2, 1), (3, 0)):
        for m, n, k in itertools.product((1, 16, 17, 63, 64, 65, 128, 129, 300, 512, 1000, 2048, 9000, 15300), (4, 64, 512, 1004, 3072, 4096, 32000),
                                         (64, 128, 192, 512, 576, 1024, 4096)):
            for ks in (1, 2, 4, 8) if kind == 2 else (1,):
                v = L.lds_variant(m, n, k, kind, ks, ragged)
                assert 0 <= v <= 7
                if v:
                    seen.add((kind, v))
                    assert m > 16 and n >= 64 and k % (chunk[v - 1] * ks) == 0 and (kind != 3 or 3 <= v <= 5)
    # output layers of 128 to 256 rows are no small products: gemm_kernel has no large tile in bf16
    assert all(L.lds_variant(m, 32000, 512, 1, 1, 0) for m in (128, 185, 256)) and not L.lds_variant(256, 2048, 512, 0, 1, 0)
    assert {v for _, v in seen} == set(range(1, 8)) and {v for kd, v in seen if kd == 3} == {3, 4, 5}


def test_splits_of_products_over_a_long_k():
    L = rules.lib()
    for m, n, k, ks in ((40, 512, 2048, 8), (64, 512, 2048, 8), (100, 512, 2048, 4), (128, 512, 2048, 4), (185, 512, 2048, 4), (256, 512, 2048, 4),
                        (300, 512, 2048, 2), (128, 1024, 4096, 4), (185, 1024, 4096, 2), (185, 512, 1024, 2), (256, 256, 1024, 4)):
        assert L.pick_ksplit(m, n, k, 0) == ks and L.kwaves_variant(m, n, k, ks) and not L.split_wm(m, n, k, ks, ks), (m, n, k)


def test_padding_does_not_choose_the_kernel_of_a_bf16_product():
    """A ragged batch has the bits of the padded one: gemm_kernel, which may add up in another order, takes both or neither."""
    L = rules.lib()
    for m, n, k, kind in itertools.product((*range(512, 1500, 20), 2440, 4500, 9000), (64, 128, 512, 1024, 1088, 2048, 3072), (64, 512, 1024, 2048, 4096), (0, 2)):
        for ks in {1, L.pick_ksplit(m, n, k, 1)} if kind == 2 else {1}:
            assert (L.lds_variant(m, n, k, kind, ks, 1) == 0) == (L.lds_variant(m, n, k, kind, ks, 0) == 0), (m, n, k, kind, ks)


def test_small_fp32_products_get_waves_that_can_share_k():
    L = rules.lib()
    waves, seen = [8, 8, 4, 4], set()
    for m, n, k, ks in itertools.product((1, 2, 17, 31, 32, 33, 64, 65, 128, 185, 256, 300, 700, 4096), (2, 4, 31, 64, 512, 1004, 2048, 4096, 32000),
                                         (32, 64, 128, 192, 256, 320, 512, 576, 1024, 1088, 4096), (1, 2, 4, 8, 16)):
        v = L.kwaves_variant(m, n, k, ks)
        assert 0 <= v <= 4
        if v:
            seen.add(v)
            assert n % 4 == 0 and k % (16 * waves[v - 1] * ks) == 0 and m * n * k <= 1.600001e9
    assert seen == {1, 2, 3, 4}


def test_small_models_leave_long_histories_to_the_launches():
    """Measured (us, launches / one workgroup a sentence): 77 / 28, 84 / 30, 84 / 89, 99 / 106, 82 / 140, 130 / 155; 89 / 58, 139 / 153."""
    L = rules.lib()
    for want, d, F, beam, batch, H, keys in ((1, 64, 256, 1, 2, 4, 800), (1, 64, 256, 1, 64, 4, 800), (0, 64, 256, 8, 2, 4, 800), (0, 64, 256, 8, 64, 4, 800),
                                             (0, 64, 256, 8, 2, 4, 2072), (0, 64, 256, 8, 64, 4, 2072), (1, 128, 512, 1, 2, 2, 800), (0, 128, 512, 1, 256, 2, 1568)):
        assert L.small_model_at(d, F, 1000, 2, beam, batch, H, keys) == want, (d, beam, batch, keys)
    for beam, batch, H in itertools.product((1, 3, 8), (1, 31, 32, 300), (1, 2, 4)):
        here = [L.small_model_at(64, 128, 1000, 3, beam, batch, H, keys) for keys in range(0, 9000, 50)]
        assert here == sorted(here, reverse=True) and here[0] == L.small_model(64, 128, 1000, 3, beam, batch)

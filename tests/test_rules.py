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

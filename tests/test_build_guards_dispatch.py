"""Register budgets of the kernels that the default options run: the lists, the
four-lane kernel, the adjoint's parts and the statistics (the compiler's report of
the build; CPU only)."""
import pytest

from paper_0908_3889_amd import build


def _resources(pattern):
    res = build.resource_usage()
    if not res:
        pytest.skip("library not built (no resource report)")
    hits = {k: {f: int(v[f]) for f in ("ScratchSize [bytes/lane]", "Occupancy [waves/SIMD]", "VGPRs Spill",
                                       "LDS Size [bytes/block]")} for k, v in res.items() if pattern in k}
    assert hits, pattern
    return hits.items()


# scratch: constants of the refill pass, stored before the loop and read there
# (two with the phase)
@pytest.mark.parametrize("kernel,waves,scratch", [
    ("integrate_list_f64ILi512ELb0E", 2, 12), ("integrate_list_f64ILi512ELb1E", 2, 20),
    ("integrate_list_f32sILi768ELb0E", 3, 0), ("integrate_list_f32sILi768ELb1E", 3, 0),
    ("integrate_list_f32xILi768ELb0E", 3, 0), ("integrate_list_f32xILi768ELb1E", 3, 0),
    ("integrate_kept_f64ILi256ELb0E", 2, 12), ("integrate_kept_f32sILi256ELb0E", 3, 0),
    ("integrate_kept_f32xILi256ELb0E", 3, 0), ("integrate_quad_f64ILi256ELb0ELb0E", 1, 0), ("integrate_quad_f64ILi256ELb0ELb1E", 1, 0),
    ("integrate_quad_f64ILi256ELb1ELb0E", 1, 0), ("adjoint_parts_kernel", 1, 0)])
def test_integration_kernels_keep_their_budget(kernel, waves, scratch):
    for name, r in _resources(kernel):
        assert r["Occupancy [waves/SIMD]"] == waves, name
        assert r["ScratchSize [bytes/lane]"] <= scratch, name


def test_block_of_the_lists_and_parts_fits_its_cu():
    for kernel, blocks in (("integrate_list_", 1), ("adjoint_parts_kernel", 4)):
        for name, r in _resources(kernel):
            assert blocks * r["LDS Size [bytes/block]"] <= 160 * 1024, name


# kernels that no scratch traffic should slow: waves on a SIMD at least
@pytest.mark.parametrize("kernel,waves", [("kde_kernel", 4), ("ks_count", 8), ("ks_scan", 4), ("ks_collect", 8),
                                          ("ks_split", 4), ("ks_solve", 4), ("ks_one", 4), ("hist_kernel", 4),
                                          ("hist2d_kernel", 4), ("pearson_part_kernel", 4), ("generate_kernel", 4)])
def test_statistics_kernels_keep_their_budget(kernel, waves):
    for name, r in _resources(kernel):
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, name
        assert r["Occupancy [waves/SIMD]"] >= waves, name


# two blocks of ks_collect share a CU: its table of up to 16,384 buckets is dynamic
def test_two_blocks_of_ks_collect_fit_a_cu():
    for name, r in _resources("ks_collect"):
        assert 2 * (r["LDS Size [bytes/block]"] + 4 * 16384) <= 160 * 1024, name

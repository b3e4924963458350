"""The counter summary's reading of a run's dispatches: which exchange a secure-ReLU call used, and which kernels belong to
which GEMM launch."""
from paper_2209_13643_amd import pmc_summary


def rows(*dispatches):
    return [(i, name, grid, kib) for i, (name, grid, kib) in enumerate(dispatches)]


def test_exchange_of_a_relu_call():
    r = rows(("k_relu_fused<2, 2, 0, false>", 131072, 100.0), ("k_copy_multi", 1, 1.0),
             ("k_relu_fused<2, 2, 0, true>", 65536, 10.0), ("k_copy_multi", 1, 1.0),
             ("k_relu_fused_msb<2, true>", 65536, 4.0), ("k_copy_multi", 1, 1.0),
             ("k_relu_fused_msb<2, false>", 65536, 2.0), ("k_copy_multi", 1, 1.0),
             ("k_relu_stage<0, 1, 0, false>", 7, 20.0), ("k_wire_words", 7, 30.0), ("k_copy_multi", 1, 1.0),
             ("k_relu_msb_stage<0, 1, true>", 7, 8.0))
    assert pmc_summary.relu_calls(r) == {("whole words", "remote store"): 100.0, ("whole words", "copy"): (10.0 + 50.0) / 2,
                                         ("sign-only", "copy"): 4.0, ("sign-only", "remote store"): (2.0 + 8.0) / 2}


def test_a_small_products_kernels_stay_with_it():
    big = ("k_limb_gemm<2, 2, true, 3, 2>", 262144, 50.0)
    r = rows(("k_open_recode<2, OpenPlanes::kFolded>", 9, 1.0), big,
             ("k_recode_mixed", 96, 1.0), ("k_sliced_gemm<false, 8>", 8192, 3.0),
             ("k_open_recode<2, OpenPlanes::kFolded>", 9, 1.0), big,
             ("k_recode_mixed", 64, 1.0), ("k_few_rows_gemm<false>", 512, 3.0),
             big,
             ("k_recode_mixed", 300, 1.0), big)
    assert pmc_summary.gemm_launches(r) == {"folded prepared call (three products)": [50.0, 50.0],
                                            "call whose recoding launch has grid 300": [50.0]}

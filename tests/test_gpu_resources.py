"""Registers, scratch and residency of the compiled kernels, as the device reports
them: what the launch configurations promise."""
import pytest
import torch

from paper_2007_01277_amd import hfuse as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    assert torch.cuda.is_available()
    H.hf_init()


@pytest.mark.parametrize("block", [256, 512, 1024])
@pytest.mark.parametrize("kind", range(H.HF_ETHASH))
def test_walk_pairs_without_a_bound_are_unbounded(kind, block):
    """vgpr_cap 0 bounds nothing, so nothing spills, and a bound of 64 registers is
    not what the unbounded kernel has."""
    i = H.hf_fused_info(kind, H.HF_ETHASH, block, 0)
    assert i["spill_bytes"] == 0, i["spill_bytes"]
    assert i["vgprs"] > 64


@pytest.mark.parametrize("block", [256, 512])
def test_sha256d_next_to_walks_keeps_six_wavefronts_per_simd(block):
    assert H.hf_fused_info(H.HF_SHA256D, H.HF_ETHASH, block, 0)["waves_per_simd"] >= 6


@pytest.mark.parametrize("block", [256, 512, 1024])
@pytest.mark.parametrize("kind", [H.HF_INT_MIX, H.HF_IM2COL, H.HF_LDS_HIST, H.HF_UPSAMPLE, H.HF_SHA256D, H.HF_BLAKE2B])
def test_statistics_bound_to_64_registers_do_not_spill(kind, block):
    i = H.hf_fused_info(H.HF_BN_STATS, kind, block, 64)
    assert i["spill_bytes"] == 0 and i["vgprs"] <= 64


@pytest.mark.parametrize("kind", [H.HF_INT_MIX, H.HF_IM2COL, H.HF_BLAKE2B])
def test_histogram_pairs_fit_two_workgroups_of_1024_on_a_cu(kind):
    assert H.hf_fused_info(min(kind, H.HF_LDS_HIST), max(kind, H.HF_LDS_HIST), 1024, 0)["wg_per_cu"] == 2


def test_upsample_fits_eight_wavefronts_on_a_simd():
    for block in (256, 512, 1024):
        assert H.hf_solo_info(H.HF_UPSAMPLE, block)["waves_per_simd"] == 8
        assert H.hf_fused_info(H.HF_LDS_HIST, H.HF_UPSAMPLE, block, 0)["waves_per_simd"] == 8

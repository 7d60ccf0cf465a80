"""Register budget of the FP32 network's kernels on the half-precision matrix cores, of the encoders and heads that run
apart, of the crop and of the voxel MLPs (CPU only): none spills a vector register."""

import pytest

from test_kernel_resources import _spills

# source file -> (symbol fragments, kernels they name)
KERNELS = {
    "net_split.hip": [("encoder_split_kernel", 4), ("chain_features_kernel", 4), ("head_split_kernel", 4),
                      ("repack_kernel", 1)],
    "head_bf16.hip": [("head_bf16_kernelILi256ELi512E", 2)],
    "fused.hip": [("fused_bf16_kernelILi128ELi256ELi512ELb1ELb0ELb1E", 1)],            # encoder alone
    "fused_fp8.hip": [("encoder_head_fp8_kernelILi128ELi256ELi512ELb0ELb1E", 1)],      # encoder alone
    "crop.hip": [("crop_kernel", 12), ("pair_setup_kernel", 1)],
    "clusters.hip": [("cluster_kernel", 1)],
    "grad.hip": [("head_backward_kernel", 2), ("pose_kernel", 2), ("head_train_kernel", 2), ("train_partials_kernel", 2),
                 ("train_reduce_kernel", 2)],
    "voxel.hip": [("point_mlp_kernel", 1), ("mlp_kernelENS0_8PairArgs", 1), ("select_kernel", 1), ("conv_kernelILi", 2)],
}


@pytest.mark.parametrize("src", sorted(KERNELS))
def test_no_vector_spills(src, tmp_path):
    found = _spills(src, tmp_path)
    for frag, count in KERNELS[src]:
        hits = {k: v for k, v in found.items() if frag in k}
        assert len(hits) == count, f"{frag} in the metadata of {src}: {sorted(found)}"
        for k, (vgpr, spill) in hits.items():
            print(f"{k}: {vgpr} VGPRs, {spill} spilled")
            assert spill == 0, f"{k} spills {spill} VGPRs ({vgpr} VGPRs)"

"""Which launch of a profile computes what, from the mangled kernel names."""
from paper_2504_03871_amd import profsummary as P

TN = "_ZN3moe16gemm_bf16_kernelIDF16bLi2ELi5ELb0ELb0ELi256ELi256ELi2ELi4EEEvNS_8GemmArgsE.kd"
DH_PAIR = "_ZN3moe21gemm_bf16_pair_kernelIDF16bLi1ELi3ELb0ELi256ELi2ELi5ELi256ELi256ELi2ELi4EEEvNS_8GemmArgsES2_i.kd"
DX_PAIR = "_ZN3moe21gemm_bf16_pair_kernelIDF16bLi1ELi0ELb0ELi160ELi2ELi5ELi256ELi256ELi2ELi4EEEvNS_8GemmArgsES2_i.kd"
F32_DX_PAIR = "_ZN3moe20gemm_f32_pair_kernelILi0ELb1ELi64ELi64EEEvNS_8GemmArgsES1_i.kd"


def test_gradients_with_a_launch_of_their_own():
    assert P.gradient_launches([TN]) == ["dw2_bwd", "dw1_bwd"]
    assert P.gradient_launches([DH_PAIR, TN]) == ["dw1_bwd"]
    assert P.gradient_launches([DX_PAIR, TN]) == P.gradient_launches([F32_DX_PAIR]) == ["dw2_bwd"]
    assert P.gradient_launches([DH_PAIR, DX_PAIR]) == []


def test_roles():
    assert P.gemm_role(TN, "dw2_bwd")[0] == "dw2_bwd" and P.gemm_role(TN)[0] == "dw1_bwd"
    assert P.gemm_role(DH_PAIR)[0] == "dh_bwd" and P.gemm_role(DX_PAIR)[0] == P.gemm_role(F32_DX_PAIR)[0] == "dx_bwd"
    assert P.gemm_role("_ZN3moe14combine_kernelIDF16bLi2ELi4EEEvPKT_.kd") == (None, "")

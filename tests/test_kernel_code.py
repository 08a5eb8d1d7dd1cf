"""Properties of the compiled kernels that no result shows."""
import pytest

from tests import kernel_code


@pytest.mark.parametrize("form", ["IDF16bLi256ELi1", "IDF16bLi256ELi2", "IfLi256ELi1", "IfLi256ELi2"])
def test_norm_backward_reads_the_statistics_through_the_scalar_unit(form):
    """A row's mean and rstd are single floats.  As vector loads they are younger than the next rows' loads, and waiting for them waits
    for those too (memory operations are counted in order)."""
    for name in kernel_code.kernels("ln_bwd_kernel" + form):
        code = kernel_code.instructions(name)
        assert any(i.startswith("global_load_dwordx4") for i in code), name
        assert not [i for i in code if i.split()[0] in ("global_load_dword", "flat_load_dword", "buffer_load_dword")], name


@pytest.mark.parametrize("kernel", ["attn_dq_kernelILi", "attn_fwd8_kernelILi", "attn_fwd_kernelILi", "attn_dkv_narrow_kernelILi", "attn_bwd_small_kernelILi", "attn_f32_bwd_kernelILi", "cross_entropy_row_kernelI",
                                    "ln_bwd_kernel", "gemm_mfma_kernel", "gemm_ring_kernel", "grad_group_kernel"])
def test_no_register_is_spilled(kernel):
    for name, k in kernel_code.kernels(kernel).items():
        assert k[".vgpr_spill_count"] == 0, (name, k[".vgpr_spill_count"])


def test_no_buffer_access_has_a_scalar_offset():
    """A buffer's range check covers the offset in the vector register and the immediate one.  The kernels rely on it for rows and columns past the end."""
    for name in kernel_code.kernels(""):
        for i in kernel_code.instructions(name):
            words = i.replace(",", " ").split()
            if words[0].startswith("buffer_") and "offen" in words:
                assert words[words.index("offen") - 1] == "0", (name, i)


@pytest.mark.parametrize("kernel", ["attn_fwd_kernelILi", "attn_dq_kernelILi", "attn_dkv_narrow_kernelILi", "attn_bwd_small_kernelILi"])
def test_staged_tiles_begin_at_the_start_of_lds(kernel):
    """These kernels turn from one buffer to the other by an XOR of the address, so their dynamic LDS has to begin at 0: no static LDS before it."""
    for name, k in kernel_code.kernels(kernel).items():
        assert k[".group_segment_fixed_size"] == 0, name

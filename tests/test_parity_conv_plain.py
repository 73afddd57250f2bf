"""The convolution kernels that need no workspace, which is what the plain C entries (sws_conv1d, sws_conv2d and their adjoints) run on: the
tests of the forward calls and of the adjoints again, with no memory lent."""
import pytest

from test_parity_conv import (B, test_cfg4_conv2d_full_size, test_conv1d_dense, test_conv1d_dense_dilated_and_long_kernels,  # noqa: F401
                              test_conv1d_dense_split_operands, test_conv1d_dense_split_operands_carry_every_bit, test_conv1d_dense_strided,
                              test_conv1d_few_channels_on_the_vector_alu, test_conv1d_integer_valued_bit_exact, test_conv2d,
                              test_conv2d_any_channel_count_and_wide_kernels, test_conv2d_chunks_of_kernel_rows,
                              test_conv2d_integer_valued_bit_exact, test_conv2d_kernel_selection_paths, test_conv2d_strided,
                              test_split_operand_kernel_carries_every_bit, test_streaming_kernel_1d, test_streaming_kernel_3x3)
from test_parity_conv_grad import (test_conv1d_adjoints_short_rows, test_conv1d_adjoints_stride_2, test_conv2d_adjoints,  # noqa: F401
                                   test_conv2d_adjoints_resnet_layer_slice, test_conv2d_adjoints_row_stride_2, test_conv2d_adjoints_short_rows,
                                   test_exact_on_small_integers, test_grad_input, test_grad_weight, test_layer_shaped_dense,
                                   test_split_operand_grad_weight, test_split_operand_grad_weight_carries_every_bit,
                                   test_split_operand_grad_weight_rows_1d, test_split_operand_grad_weight_rows_2d,
                                   test_split_operand_grad_weight_rows_at_full_size_on_sampled_channels,
                                   test_split_operand_grad_weight_rows_carry_every_bit)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_workspace(B, monkeypatch):  # noqa: F811
    monkeypatch.setattr(B, "_scratch", lambda n, like, stream: (None, None, 0))

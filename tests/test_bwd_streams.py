"""Where the backward pass takes its second stream, on both sides of the rule (host only; that one or two streams give the same bits is a GPU
test)."""
import pytest

import paper_2204_06514_amd as fax


@pytest.mark.parametrize("B,S,D,H,F,streams", [
    (8, 1024, 1024, 16, 4096, 1),    # weight gradients in one launch, input gradients 32 x 8 tiles of 256 x 128
    (8, 2048, 1024, 8, 4096, 2),     # in one launch beside QKV's input gradient, those of the feed-forward 64 x 16 and 64 x 4 tiles of 256 x 256: 1588 us; four launches 1649, two on one stream 1701
    (8, 512, 1024, 16, 4096, 2),     # in two launches, smaller tiles, 312 us
    (2, 1024, 1024, 8, 4096, 1),     # under 200 us, in one launch with QKV's input gradient
    (4, 777, 512, 8, 2048, 2),       # under 200 us, a fifth idle
    (4, 1024, 512, 8, 2048, 2),      # under 200 us, nothing idle, separate launches
    (8, 2048, 2048, 16, 8192, 2),    # whole rounds only without the weight gradients
    (3, 2500, 1024, 16, 4096, 2),    # input gradients of 240 tiles
    (2, 2048, 4096, 32, 16384, 1)])  # whole rounds throughout
def test_second_stream_where_rounds_leave_places(B, S, D, H, F, streams):
    for flags, want in ((0, streams), (fax.FAX_FLAG_SINGLE_STREAM, 1), (fax.FAX_FLAG_TP_PARTIAL, streams)):
        assert fax.fax_block_bwd_streams(fax.block_dims(B, S, D, H, D // H, F, fax.FAX_BF16, fax.FAX_GELU_TANH, 1e-5, flags)) == want


@pytest.mark.parametrize("B,S,D,H,streams", [(2, 64, 128, 4, 1), (2, 256, 512, 8, 1), (1, 256, 1024, 16, 1), (3, 300, 512, 8, 2), (1, 777, 768, 12, 2), (4, 512, 1024, 16, 2)])
def test_second_stream_of_fp32_blocks_by_the_estimate_of_their_kernel(B, S, D, H, streams):
    d = lambda flags: fax.block_dims(B, S, D, H, D // H, 4 * D, fax.FAX_F32, fax.FAX_GELU_TANH, 1e-5, flags)  # noqa: E731
    assert fax.fax_block_bwd_streams(d(0)) == streams and fax.fax_block_bwd_streams(d(fax.FAX_FLAG_SINGLE_STREAM)) == 1

"""The distillation loss over few and many vocabulary chunks: which logits of the first pass are still there in the second
(the last two chunks' on the fused path, the last one's otherwise) depends on the number of chunks and on their width."""
import pytest

from test_gpu_section import _kd_loss_standalone

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,ht,hs", [("bf16", 128, 64), ("bf16", 72, 40), ("fp32", 72, 40)])   # fused, not fused, fp32
@pytest.mark.parametrize("vocab,chunk", [(256, 512), (256, 256), (256, 128), (328, 128), (648, 128), (40, 8), (64, 16), (296, 72)])
def test_chunk_counts_and_widths(dtype, ht, hs, vocab, chunk):
    _kd_loss_standalone(dtype, vocab, chunk, 45, ht, hs, 1.5, 0)

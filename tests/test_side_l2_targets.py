"""Which targets the L2 loss reads straight from memory (CPU): those whose memory
holds their values as the image's does."""
import pytest
import torch

from paper_2507_23189_amd import autograd as A

IMAGE = torch.zeros((6, 5), dtype=torch.float64)
RAND = torch.rand((6, 5), dtype=torch.float64)


@pytest.mark.parametrize("target, reads", [
    (RAND, True), (torch.rand((12, 5), dtype=torch.float64)[6:], True), (RAND.clone().requires_grad_(), True),
    (RAND.float(), False), (RAND.t().contiguous().t(), False), (RAND[:1].expand(6, 5), False), (RAND[0], False),
    (torch.nn.Parameter(RAND), False), (RAND.to_sparse(), False), (RAND.tolist(), False), (0.25, False),
    (torch._neg_view(RAND), False), (torch._efficientzerotensor((6, 5), dtype=torch.float64), False),
    (RAND.to("meta"), False),
], ids=["image", "rows", "leaf", "float32", "columns", "broadcast", "row", "parameter", "sparse", "list", "number", "negated",
        "zero", "meta"])
def test_targets_read_from_memory(target, reads):
    assert A._reads_as(target, IMAGE) is reads


def test_one_pixel_of_a_conjugate():
    z = torch.complex(RAND[:1, :1], RAND[:1, :1]).conj().imag   # contiguous, its memory of the other sign
    assert not A._reads_as(z, IMAGE[:1, :1]) and A._reads_as(z.resolve_neg(), IMAGE[:1, :1])

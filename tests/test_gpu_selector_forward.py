"""Forward passes of more samples than one round of the blocks: every sample's logits are those of a small batch."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [31, 32, 33, 16383, 16384, 16385, 32769, 65536])
def test_logits_do_not_depend_on_the_batch(batch):
    import torch
    import paper_1804_06926_amd as tc
    from paper_1804_06926_amd import selector
    assert selector.load_default()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch)
    x = torch.rand((batch, 6), generator=gen, device="cuda")
    z = tc.selector_forward(x)
    for a in range(0, batch, 8192):   # 256 rounds: one per block
        assert torch.equal(z[a:a + 8192], tc.selector_forward(x[a:a + 8192].contiguous()))

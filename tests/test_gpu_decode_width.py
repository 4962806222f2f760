"""The decode step where its block width changes (two rows per CU) and at its
grid-stride limit: rows that are rewritten next to rows that are not."""
import pytest
import torch

from paper_2608_24658_amd import parason as PX

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("per_cu,more", [(2, 0), (2, 1), (8, 0), (8, 3)])
@pytest.mark.parametrize("vocab", [997, 12288])
def test_block_widths(dtype, per_cu, more, vocab):
    batch = torch.cuda.get_device_properties(0).multi_processor_count * per_cu + more
    tags = list(range(vocab - 12, vocab))
    h = PX.Parason(tags)
    states = PX.decode_init(batch, "cuda")
    x = torch.randn(batch, vocab, device="cuda").to(dtype)
    think = tags[0]
    got = h.decode_step(states, x.clone())
    want = torch.full_like(x, float("-inf"))
    want[:, think] = x[:, think]
    assert torch.equal(got, want)  # only <Think> may come first
    tok = torch.full((batch,), think, dtype=torch.int32, device="cuda")
    tok[1::3] = -1
    got = h.decode_step(states, x.clone(), tok)
    body = x.clone()  # in the body: text, <Parallel>, </Think>
    for c, t in enumerate(tags):
        if c not in (1, 2):
            body[:, t] = float("-inf")
    body[1::3] = want[1::3]
    assert torch.equal(got, body)

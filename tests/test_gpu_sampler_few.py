"""The accept rule with few sequences (decisions taken inside the mass pass) against the same
sequences in one large batch (decisions in a launch of their own): bit for bit, at vocabularies
of one partial chunk to several, with aligned and unaligned rows, with and without q, k = 0, and
past one batch of accept rows; logits with infinities and far apart among them."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,k,with_q", [
    (5, 0, False), (300, 2, True), (8192, 4, True), (8193, 3, False), (20004, 15, True), (24577, 4, True),
    (8200, 17, True),
])
def test_few_equals_batch(molt_lib, V, k, with_q):
    print(f"case V={V} k={k} q={with_q}", flush=True)
    B = 200                                              # 200 chunks and more: the batch path
    g = torch.Generator(device="cuda").manual_seed(V + k)
    logits = 3.0 * torch.randn(B, k + 1, V, generator=g, device="cuda")
    logits[3] *= 40.0                                    # p underflows for most tokens
    logits[5, :, 1:] = -float("inf")                     # one token has all the mass
    logits[7, :, ::2] = -float("inf")
    q = torch.softmax(logits[:, :k] + torch.randn(B, k, V, generator=g, device="cuda"), -1)
    drafts = torch.stack([torch.multinomial(q[:, i] + 1e-30, 1, generator=g)[:, 0] for i in range(k)], 1).int() \
        if k else torch.zeros(B, 0, dtype=torch.int32, device="cuda")
    u = torch.rand(B, k + 1, generator=g, device="cuda")
    qa = q.contiguous() if with_q and k else None
    big = molt_lib.spec_accept(logits, drafts.contiguous(), u, qa)
    for b in (0, 1, 3, 5, 7, 64, 199):
        one = molt_lib.spec_accept(logits[b:b + 1].contiguous(), drafts[b:b + 1].contiguous(),
                                   u[b:b + 1].contiguous(), None if qa is None else qa[b:b + 1].contiguous())
        for x, y in zip(big, one):
            x = x[b:b + 1]
            assert torch.equal(torch.nan_to_num(x.double(), nan=7e9), torch.nan_to_num(y.double(), nan=7e9)), b

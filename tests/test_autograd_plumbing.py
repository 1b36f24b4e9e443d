"""The autograd wrapper without a GPU: what reaches the library object's backward."""
import torch

import paper_2508_18224_amd as nsa


class _Recorder:
    """Stands in for SelAttention: remembers the gradient it is handed."""

    def forward(self, q, k, v, idx, cu, rebuild_index=True):
        return q * 2, q[..., 0] * 0

    def backward(self, q, k, v, o, lse, do, cu):
        self.do = do
        return do * 2, torch.zeros_like(k), torch.zeros_like(v)


class _Cut(torch.autograd.Function):
    """Passes a value on and no gradient back."""

    @staticmethod
    def forward(ctx, x):
        return x.clone()

    @staticmethod
    def backward(ctx, g):
        return None


def test_output_without_gradient_gives_zero_gradients():
    q, k, v = (torch.ones(4, 2, 8, requires_grad=True) for _ in range(3))
    attn = _Recorder()
    o, lse = nsa.selected_attention(q, k, v, None, attn)
    _Cut.apply(o).sum().backward()
    assert torch.equal(attn.do, torch.zeros_like(o)) and torch.equal(q.grad, torch.zeros_like(q))
    assert not lse.requires_grad


def test_strided_gradient_arrives_contiguous():
    q, k, v = (torch.ones(4, 2, 8, requires_grad=True) for _ in range(3))
    attn = _Recorder()
    o, _ = nsa.selected_attention(q, k, v, None, attn)
    o.backward(torch.arange(64.0).view(8, 2, 4).transpose(0, 2))
    assert attn.do.is_contiguous() and torch.equal(q.grad, 2 * torch.arange(64.0).view(8, 2, 4).transpose(0, 2))

"""The tile lists do not depend on how the rows are launched: the totals of the
workgroups added up by every workgroup, or scanned first for many.  The
same block mask is expanded for all KV heads in one call and in slices of the
heads (without the random rescue, whose hash takes the head's number)."""
import pytest
import torch

from paper_2605_12193_amd import bfla

pytestmark = pytest.mark.gpu


def _expand(n, h_kv, mask, prm):
    prob = bfla.Problem(n, n, h_kv, h_kv, 64)
    buf = bfla.Buffers(prob, prm)
    buf.row_ptr.fill_(-1)
    bfla.bfla_expand_rescue(prob, prm, mask, buf.row_ptr, buf.cols, buf.ws_expand)
    torch.cuda.synchronize()
    return buf.row_ptr, buf.cols[:int(buf.row_ptr[-1])]


# (tokens, KV heads in one call, heads per slice): one row; 16 rows a head, two
# whole workgroups; 65 rows a head; 516 rows a head, 33024 rows (4128 totals:
# scanned) in slices of 16512 (2064: added up); rows of 9 ballot words
@pytest.mark.parametrize("n,h_kv,per", [(64, 1, 1), (1000, 9, 1), (4160, 3, 1), (33000, 64, 32),
                                        (36000, 2, 1)])
def test_lists_are_the_same_in_every_launch_form(n, h_kv, per):
    gen = torch.Generator(device="cuda").manual_seed(n + h_kv)
    prm = bfla.params(rho=0.0, seed=5)
    lb = -(-n // 128)
    mask = (torch.rand(h_kv, lb, lb, device="cuda", generator=gen) < 0.1).to(torch.uint8)
    ptr, cols = _expand([n], h_kv, mask, prm)
    t_q = -(-n // 64)
    at = 0
    for h in range(0, h_kv, per):
        p, c = _expand([n], per, mask[h:h + per].contiguous(), prm)
        lo, hi = h * t_q, (h + per) * t_q
        assert torch.equal(ptr[lo:hi + 1] - ptr[lo], p)
        assert torch.equal(cols[at:at + c.numel()], c)
        at += c.numel()
    assert at == cols.numel() == int(ptr[-1]) and int(ptr[0]) == 0


def test_lists_over_several_launch_groups():
    """40 requests (two launch groups) in one call and one by one."""
    gen = torch.Generator(device="cuda").manual_seed(1)
    prm = bfla.params(rho=0.0, seed=5)
    n = [64 * (1 + 7 * i % 11) - i for i in range(40)]
    masks = [(torch.rand(2 * (-(-x // 128)) ** 2, device="cuda", generator=gen) < 0.2).to(torch.uint8)
             for x in n]
    ptr, cols = _expand(n, 2, torch.cat(masks), prm)
    row = 0
    for x, m in zip(n, masks):
        p, c = _expand([x], 2, m, prm)
        lo = int(ptr[row])
        assert torch.equal(ptr[row:row + p.numel()] - lo, p)
        assert torch.equal(cols[lo:lo + c.numel()], c)
        row += p.numel() - 1

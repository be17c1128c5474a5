"""Launches of few rows and heads deal a tile's keys to 2, 4 or 8 groups of the workgroup's waves (attn_stream16.hip);
the groups' results meet in LDS.  Where that can go wrong: shares of unequal length, fewer kblocks than groups, a last
kblock of one key, a last tile of one row, a score far above its own group's reference.  The launch rule gives the
small shapes here the largest grouping a head_dim has (8 groups at 64, 4 at 128); 24 heads of 1170 rows get two."""
import pytest
import torch

from paper_2509_22622_amd import binding as B

pytestmark = pytest.mark.gpu


def _reference(q, k, v):
    """[rows, H, D] in 64 bits."""
    q, k, v = (x.double().transpose(0, 1) for x in (q, k, v))
    w = torch.softmax(torch.stack([a @ b.T.contiguous() for a, b in zip(q, k)]) * q.shape[-1] ** -0.5, -1)
    return torch.stack([a @ b for a, b in zip(w, v)]).transpose(0, 1)


def _check(heads, head_dim, n_q, n_keys, seed, spoil=None):
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = (torch.empty((n, heads, head_dim), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
               for n in (n_q, n_keys, n_keys))
    if spoil is not None:
        spoil(q, k)
    prompt = B.Prompt(1, heads, head_dim, n_keys)
    prompt.recache(0, k, v)
    out = torch.full_like(q, 7.0)
    prompt.cross_attn(0, q, out)
    torch.cuda.synchronize()
    prompt.close()
    want = _reference(q, k, v)
    err = (out.double() - want).norm() / want.norm()
    return out, want, float(err)


@pytest.mark.parametrize("heads, head_dim", [(2, 64), (3, 128)])
@pytest.mark.parametrize("n_keys", [1, 31, 33, 64, 97, 128, 225, 256, 257, 289, 511, 1000])
@pytest.mark.parametrize("n_q", [1, 33, 64, 95])
def test_shares_of_every_length(heads, head_dim, n_q, n_keys):
    """bf16 operands and weights: half a unit in the last place (2^-9) on q', on the weights and on the result, in
    quadrature about 2.9e-3; up to 5e-3 where few keys leave nothing to average over."""
    _, _, err = _check(heads, head_dim, n_q, n_keys, 1000 * n_q + n_keys)
    assert err <= 5e-3


@pytest.mark.parametrize("n_keys", [65, 384, 399])
def test_two_groups(n_keys):
    _, _, err = _check(24, 128, 1170, n_keys, n_keys)
    assert err <= 5e-3


@pytest.mark.parametrize("heads, head_dim, n_q", [(2, 64, 70), (3, 128, 70), (24, 128, 1170)])
@pytest.mark.parametrize("at", [3, 300, 511])
def test_a_score_far_above_one_groups_reference(heads, head_dim, n_q, at):
    """Key `at` is 40 times query 5: its logit exceeds every other of that row by some 40 sqrt(D), beyond what a fixed
    reference holds, and the whole weight of the row lies in one group."""
    def spoil(q, k):
        k[at] = 40 * q[5]

    out, want, _ = _check(heads, head_dim, n_q, 512, at, spoil)
    assert bool(torch.isfinite(out).all())
    row = want[5]
    assert float((out[5].double() - row).norm() / row.norm()) <= 2.0 ** -8

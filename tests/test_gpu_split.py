"""Items shared by several slots of a workgroup (few items, many compute units) vs the reference."""

import numpy as np
import pytest

import oracle
from helpers import compare, to_bits
from workloads import pack_rows

pytestmark = pytest.mark.gpu

CASES = [
    # (B, H, N, d, blk_q, blk_k, p, seed): p = chance of a block
    (1, 2, 1000, 128, 128, 128, 0.5, 1),    # two parts, ragged last block
    (2, 1, 1030, 64, 128, 128, 0.3, 2),     # the last query and key block hold 6 tokens
    (1, 3, 700, 128, 128, 64, 0.4, 3),
    (1, 3, 700, 64, 128, 64, 0.4, 4),
    (1, 2, 1000, 128, 64, 64, 0.5, 5),      # four parts
    (2, 2, 577, 64, 64, 64, 0.2, 6),        # four parts, a last block of one token
    (1, 2, 2050, 64, 64, 128, 0.3, 7),
    (1, 2, 1100, 128, 64, 128, 0.3, 8),     # too large for LDS: never shared
    (1, 8, 4096, 64, 128, 128, 0.05, 9),    # 256 items: the last shape with two parts
    (1, 9, 3700, 64, 128, 128, 0.05, 10),   # 261 items: not shared
    (1, 8, 2048, 64, 64, 64, 0.08, 11),     # 256 items of 64 rows: the last with four parts
    (1, 9, 1850, 64, 64, 64, 0.08, 12),     # 261: two parts
    (1, 16, 2048, 128, 64, 64, 0.05, 13),   # 512: the last with two parts
    (1, 19, 1750, 64, 64, 64, 0.08, 14),    # 532: not shared
    (1, 2, 480, 128, 64, 64, 0.5, 15),      # 8 key blocks: the shortest rows shared
    (1, 2, 440, 128, 64, 64, 0.5, 16),      # 7: not shared
]


@pytest.mark.parametrize("B,H,N,d,blk_q,blk_k,p,seed", CASES)
def test_shared_items_match_reference(B, H, N, d, blk_q, blk_k, p, seed):
    import torch
    from paper_2606_23019_amd import binding
    rng = np.random.default_rng(seed)
    n_qb, n_kb = -(-N // blk_q), -(-N // blk_k)
    mask = rng.random((H, n_qb, n_kb)) < p
    # rows of 0, 1, 2, 3 and 5 blocks: parts without a block; one row with all
    for u, c in enumerate((0, 1, 2, 3, 5)):
        mask[0, u % n_qb] = False
        mask[0, u % n_qb, rng.choice(n_kb, c, replace=False)] = True
    mask[-1, -1] = True
    packed = pack_rows(mask)
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = (torch.randn((B, H, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))
    out, lse = binding.bsattn_fwd(q, k, v, packed, blk_q, blk_k)
    ref = oracle.attention(to_bits(q), to_bits(k), to_bits(v), packed, blk_q, blk_k, d ** -0.5)
    compare(out.float().cpu().numpy(), lse.cpu().numpy(), *ref)
    # the same bits through the plan, in fp32 before rounding, on [B, N, H, d], and in any order
    plan = binding.Plan(packed, B, H, N, blk_q, blk_k)
    o2, l2 = plan(q, k, v)
    o3, l3 = plan.fwd_f32out(q, k, v)
    o4, l4 = binding.bsattn_fwd_bnhd(*(x.transpose(1, 2).contiguous() for x in (q, k, v)), packed,
                                     blk_q, blk_k)
    counts, lists = binding.mask_prepass(packed, H, n_qb, n_kb)
    order = torch.from_numpy(rng.permutation(B * H * n_qb).astype(np.int32)).cuda()
    o5, l5 = binding.bsattn_fwd_prepared(q, k, v, counts, lists, order, blk_q, blk_k)
    for o, l in ((o2, l2), (o3.bfloat16(), l3), (o4.transpose(1, 2), l4), (o5, l5)):
        assert torch.equal(o, out) and torch.equal(l, lse)


@pytest.mark.parametrize("N,blk,d", [(1000, 128, 128), (1000, 64, 64)])
def test_part_of_infinitely_low_logits_adds_nothing(N, blk, d):
    # keys of the last blocks, a part of their own, have logits of -inf; the
    # others are what is left
    import torch
    from paper_2606_23019_amd import binding
    g = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn((1, 1, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))
    q[..., 0] = q[..., 0].abs() + 1.0
    n_kb = -(-N // blk)
    kept = n_kb // 2
    k[:, :, kept * blk:, 0] = -torch.inf
    rows = np.ones((1, n_kb, n_kb), dtype=bool)
    out, lse = binding.bsattn_fwd(q, k, v, pack_rows(rows), blk, blk)
    rows[:, :, kept:] = False
    kf = k.clone()
    kf[:, :, kept * blk:] = 0.0
    ref = oracle.attention(to_bits(q), to_bits(kf), to_bits(v), pack_rows(rows), blk, blk, d ** -0.5)
    compare(out.float().cpu().numpy(), lse.cpu().numpy(), *ref)


def _attend(call, q, k, v, rows, blk):
    from paper_2606_23019_amd import binding
    B, H, N, _ = q.shape
    if call == "dense":
        return binding.dense_attn_fwd(q, k, v, blk)
    if call == "oneshot":  # walks the mask where one item fills a workgroup
        return binding.bsattn_fwd(q, k, v, pack_rows(rows), blk, blk)
    return binding.Plan(pack_rows(rows), B, H, N, blk, blk)(q, k, v)


NON_FINITE = [
    # (call, H, N, d, blk): two and four parts, off the mask, off the list and maskless
    ("oneshot", 1, 1000, 128, 128), ("plan", 1, 1000, 128, 128), ("dense", 1, 1000, 128, 128),
    ("oneshot", 1, 2050, 64, 64), ("plan", 1, 2050, 64, 64), ("dense", 1, 2050, 64, 64),
    ("plan", 9, 2050, 64, 64),
    ("dense", 57, 1100, 64, 128),  # a shared last round
    ("plan", 57, 1100, 64, 128),   # not shared
]


@pytest.mark.parametrize("call,H,N,d,blk", NON_FINITE)
def test_nan_in_any_part_reaches_the_output(call, H, N, d, blk):
    # a run of key blocks with NaN keys, or with NaN values that weigh nothing: parts of their
    # own, or the first, middle or last blocks of a part
    import torch
    n = -(-N // blk)
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn((1, H, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))
    q[..., 0] = 1.0
    rng = np.random.default_rng(N)
    for at, end in ((0, 1), (1, 2), (n // 2, n // 2 + 1), (n - 1, n), ((n + 1) // 2, n),
                    (0, (n + 1) // 2), (n - n // 4, n)):
        rows = np.ones((H, n, n), dtype=bool)
        if call != "dense":
            others = rng.permutation(np.delete(np.arange(n), np.arange(at, end)))
            rows[:, 1:5] = False
            rows[:, 1, list(others[:3]) + [at]] = True  # four blocks, one of them bad
            rows[:, 2, [others[0], at]] = True          # two
            rows[:, 3, at] = True                       # alone
            rows[:, 4, others] = True                   # none of them bad
        hit = np.repeat(rows[0, :, at:end].any(-1), blk)[:N]
        keys = slice(at * blk, min(end * blk, N))
        clean, clean_lse = _attend(call, q, k, v, rows, blk)
        bad = k.clone()
        bad[:, :, keys] = torch.nan
        out, lse = _attend(call, q, bad, v, rows, blk)
        on = torch.from_numpy(hit).cuda()
        assert torch.isnan(out[:, :, on]).all() and not torch.isfinite(lse[:, :, on]).any(), at
        assert torch.equal(out[:, :, ~on], clean[:, :, ~on])
        assert torch.equal(lse[:, :, ~on], clean_lse[:, :, ~on])
        # a channel of NaN values: 0 times NaN, whatever the block's weight
        low = k.clone()
        low[:, :, keys, 0] = -2e4
        bad = v.clone()
        bad[:, :, keys, 3] = torch.nan
        out, _ = _attend(call, q, low, bad, rows, blk)
        want, _ = _attend(call, q, low, v, rows, blk)
        assert torch.isnan(out[:, :, on, 3]).all(), at
        bad_at = torch.isnan(out)
        bad_at[:, :, on, 3] = False
        assert not bad_at.any()
        assert torch.equal(out[..., 4:], want[..., 4:])


@pytest.mark.parametrize("call,H,N,d,blk", NON_FINITE)
def test_any_block_of_infinitely_low_logits_but_the_first_adds_nothing(call, H, N, d, blk):
    import torch
    n = -(-N // blk)
    g = torch.Generator(device="cuda").manual_seed(N + 1)
    q, k, v = (torch.randn((1, H, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))
    q[..., 0] = q[..., 0].abs() + 1.0
    heads = [0, H - 1]
    for at in sorted({1, n // 4, n // 2, n - 2, n - 1}):
        rows = np.ones((H, n, n), dtype=bool)
        keys = slice(at * blk, min((at + 1) * blk, N))
        low = k.clone()
        low[:, :, keys, 0] = -torch.inf
        out, lse = _attend(call, q, low, v, rows, blk)
        rows = rows[heads]
        rows[:, :, at] = False
        low[:, :, keys] = 0.0
        ref = oracle.attention(*(to_bits(x[:, heads]) for x in (q, low, v)), pack_rows(rows), blk,
                               blk, d ** -0.5)
        compare(out[:, heads].float().cpu().numpy(), lse[:, heads].cpu().numpy(), *ref)


def test_wide_tiles_of_the_maskless_path_match_reference():
    # blocks of 64 that would run unshared take 128 x 128 tiles from 512 tokens on
    import torch
    from paper_2606_23019_amd import binding
    for (B, H, N, d) in ((2, 33, 515, 64), (1, 60, 640, 128), (1, 66, 511, 64)):
        g = torch.Generator(device="cuda").manual_seed(N)
        q, k, v = (torch.randn((B, H, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))
        out, lse = binding.dense_attn_fwd(q, k, v, 64)
        n = -(-N // 64)
        ones = pack_rows(np.ones((H, n, n), dtype=bool))
        ref = oracle.attention(to_bits(q), to_bits(k), to_bits(v), ones, 64, 64, d ** -0.5)
        compare(out.float().cpu().numpy(), lse.cpu().numpy(), *ref)


@pytest.mark.parametrize("B,H,N,d,blk", [
    (1, 57, 1100, 64, 128),    # 513 items, 65 places an XCD: one round and one shared place
    (1, 57, 1030, 128, 64),    # the same by way of 128 x 128 tiles, ragged
    (2, 48, 1024, 64, 128),    # 96 places: the longest shared rest
    (1, 97, 961, 64, 128),     # 97: not shared
    (1, 74, 896, 64, 128),     # 65 places, rows of 7 key blocks: not shared
])
def test_shared_last_round_of_the_maskless_path(B, H, N, d, blk):
    import torch
    from paper_2606_23019_amd import binding
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn((B, H, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))
    out, lse = binding.dense_attn_fwd(q, k, v, blk)
    n = -(-N // 128)
    ones = pack_rows(np.ones((H, n, n), dtype=bool))
    ref = oracle.attention(to_bits(q), to_bits(k), to_bits(v), ones, 128, 128, d ** -0.5)
    compare(out.float().cpu().numpy(), lse.cpu().numpy(), *ref)


@pytest.mark.parametrize("H,N,d,blk_q,blk_k,p", [
    (1, 16400, 64, 128, 64, 0.03),    # rows of 5 words, the last of one block
    (1, 32768, 128, 128, 64, 0.02),   # 8 full words: the longest rows walked off the mask
    (1, 32768, 64, 128, 128, 0.01),   # 4 words, many of them empty
    (1, 8250, 128, 64, 64, 0.3),      # four parts, 3 words
    (1, 16384, 64, 64, 128, 0.05),    # four parts, 2 words
    (3, 4100, 128, 128, 128, 0.5),
])
def test_walk_off_the_mask_gives_the_bits_of_the_list(H, N, d, blk_q, blk_k, p):
    # one-shot calls of these shapes scan the mask rows in the attention kernel; a plan
    # walks the pre-pass's lists.  Bits past the last key block do not count.
    import torch
    from paper_2606_23019_amd import binding
    rng = np.random.default_rng(N + d)
    n_qb, n_kb = -(-N // blk_q), -(-N // blk_k)
    mask = rng.random((H, n_qb, n_kb)) < p
    for u, at in enumerate(([], [0], [n_kb - 1], [0, n_kb - 1], [n_kb // 2], list(range(n_kb)))):
        mask[0, u] = False
        mask[0, u, at] = True
    mask[0, 6] = np.arange(n_kb) >= n_kb // 2
    packed = pack_rows(mask)
    noisy = packed.copy()
    if n_kb % 64:
        noisy[..., -1] |= np.uint64((2 ** 64 - 1) ^ (2 ** (n_kb % 64) - 1))
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn((1, H, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))
    plan = binding.Plan(packed, 1, H, N, blk_q, blk_k)
    want, want_lse = plan.fwd_f32out(q, k, v)
    out, lse = binding.bsattn_fwd_f32out(q, k, v, noisy, blk_q, blk_k)
    assert torch.equal(out, want) and torch.equal(lse, want_lse)
    out, lse = binding.bsattn_fwd(q, k, v, noisy, blk_q, blk_k)
    assert torch.equal(out, plan(q, k, v)[0]) and torch.equal(lse, want_lse)
    t = [x.transpose(1, 2).contiguous() for x in (q, k, v)]
    out, lse = binding.bsattn_fwd_bnhd(*t, noisy, blk_q, blk_k)
    assert torch.equal(out.transpose(1, 2), plan(q, k, v)[0]) and torch.equal(lse, want_lse)


@pytest.mark.parametrize("B,H,N,d,blk,same", [
    (1, 16, 4096, 64, 128, True),     # 512 query blocks
    (2, 16, 1000, 128, 64, True),     # 512
    (1, 74, 896, 64, 128, True),      # 518, of 7 key blocks
    (1, 66, 511, 64, 64, True),       # 528, under 512 tokens
    (1, 57, 1100, 64, 128, False),    # 513 query blocks: a shared last round
    (1, 65, 512, 64, 64, False),      # 520: tiles of 128
    (1, 57, 1030, 128, 64, False),    # both
])
def test_maskless_and_all_ones_mask_on_both_sides_of_the_line(B, H, N, d, blk, same):
    # bit for bit up to 512 query blocks, or 511 (blk 64) and 896 (blk 128) tokens; beyond, to
    # within the rounding that the reference comparison allows either of them
    import torch
    from paper_2606_23019_amd import binding
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn((B, H, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))
    n = -(-N // blk)
    ones = pack_rows(np.ones((H, n, n), dtype=bool))
    out, lse = binding.dense_attn_fwd(q, k, v, blk)
    want, want_lse = binding.bsattn_fwd(q, k, v, ones, blk, blk)
    if same:
        assert torch.equal(out, want) and torch.equal(lse, want_lse)
    else:
        compare(out.float().cpu().numpy(), lse.cpu().numpy(), want.float().cpu().numpy(),
                want_lse.cpu().numpy())


@pytest.mark.parametrize("N,d,blk", [(2000, 128, 128), (1500, 64, 64)])
def test_a_head_in_calls_of_more_heads(N, d, blk):
    # shared by a rule on the whole call's shape: the same bits while the rule says the same, the
    # same result to within rounding where it does not
    import torch
    from paper_2606_23019_amd import binding
    H = 40
    n = -(-N // blk)
    mask = np.random.default_rng(N).random((H, n, n)) < 0.3
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn((1, H, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))

    def of(heads):
        o, l = binding.bsattn_fwd(*(x[:, :heads].contiguous() for x in (q, k, v)),
                                  pack_rows(mask[:heads]), blk, blk)
        return o[:, :1], l[:, :1]
    alone, few, all_ = of(1), of(4), of(H)  # 16 or 24, 64 or 96, 640 or 960 query blocks
    assert torch.equal(alone[0], few[0]) and torch.equal(alone[1], few[1])
    compare(alone[0].float().cpu().numpy(), alone[1].cpu().numpy(), all_[0].float().cpu().numpy(),
            all_[1].cpu().numpy())

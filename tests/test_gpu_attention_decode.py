"""The kernel for few queries per sequence (max_seqlen_q x query heads per key/value head <= 32) gives the bits of the
kernel for every call shape (0 differing bits), at the edges of its tiles, rounds of four tiles, splits, column groups and
channel groups; a few rows are also held against the oracle with the bars of test_gpu_attention.py."""
import numpy as np
import pytest
import torch

import gpu_util as gu
from paper_2511_17826_amd import binding as tb
from paper_2511_17826_amd import synthetic as syn
from test_gpu_attention import check_against_oracle, i32

pytestmark = pytest.mark.gpu


def both(Hq, Hkv, lens_q, lens_k, causal=True, dtype=torch.bfloat16, seed=0, poison=float("nan"), edit=None, said_q=None, ws_bytes=0):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    rnd = lambda n, h: torch.randn((n, h, 128), generator=g, device="cuda:0").to(dtype)
    Q, K, V = rnd(sum(lens_q), Hq), rnd(max(sum(lens_k), 1), Hkv), rnd(max(sum(lens_k), 1), Hkv)
    cq, ck = i32(np.cumsum([0] + list(lens_q))), i32(np.cumsum([0] + list(lens_k)))
    if edit:
        ends = np.cumsum(lens_k)
        edit(K, V, ends - np.array(lens_k), ends)
    call = tb.tbik_attention if dtype == torch.bfloat16 else tb.tbik_attention_f16
    need = ws_bytes or max(256, tb.attention_workspace_bytes(len(lens_q), max(lens_q), max(lens_k), Hq, Hkv))
    out = []
    for variant in (1, 0):
        tb.tbik_set_attention_variant(variant)
        ws = torch.full((need // 4,), poison, dtype=torch.float32, device="cuda:0")
        O = torch.full_like(Q, 7.0)
        call(Q, K, V, cq, ck, said_q if said_q and variant == 0 else max(lens_q), 128 ** -0.5, causal, out=O, max_seqlen_k=max(lens_k), workspace=ws)
        torch.cuda.synchronize()
        out.append(O.view(torch.int16).cpu())
    tb.tbik_set_attention_variant(0)
    return out


EDGES = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 191, 255, 256, 257, 300, 511, 513, 1000]


@pytest.mark.parametrize("Hq,Hkv,q", [(4, 4, 1), (8, 4, 2), (8, 2, 1), (8, 2, 3), (8, 2, 4), (8, 2, 5), (8, 2, 8), (10, 2, 1), (10, 2, 3),
                                      (32, 2, 1), (24, 1, 1), (32, 1, 1), (3, 1, 7)])
@pytest.mark.parametrize("causal", [True, False])
def test_few_queries_same_bits_at_tile_and_round_edges(Hq, Hkv, q, causal):
    lens_q = [1 + (i * 7) % q for i in range(len(EDGES))]
    lens_q[3] = q
    a, b = both(Hq, Hkv, lens_q, [max(k, 1) for k in EDGES], causal, seed=q)
    assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("batch,Hkv", [(1, 1), (3, 8), (9, 8), (17, 8), (40, 8), (70, 8)])
@pytest.mark.parametrize("causal", [True, False])
def test_splits_in_parallel_walked_and_channel_groups_same_bits(dtype, batch, Hkv, causal):
    """1 to 3 splits of 4096 keys, sequences without keys or queries among them; few items (channel groups, one workgroup
    per split and a fold) to many (splits walked)."""
    lens = [4096, 4097, 4160, 8192, 8193, 4351, 100, 0, 9000, 4095]
    lens_k = [lens[(3 * i) % len(lens)] for i in range(batch)]
    lens_q = [1] * batch
    if batch > 5:
        lens_q[5] = 0
    a, b = both(4 * Hkv, Hkv, lens_q, lens_k, causal, dtype=dtype, seed=batch)
    assert torch.equal(a, b)


@pytest.mark.parametrize("causal", [True, False])
def test_short_workspace_walks(causal):
    """A workspace of the size that the kernel for every call shape asks for (one state of 68 KiB per item where it walks the
    splits) does not hold the states of 40 sequences x 8 heads x 15 splits: the splits are walked, same bits; less is refused."""
    lens_k = [61440, 8193, 4096] + [70 + i for i in range(37)]
    lens_q = [1] * 40
    required = (40 * 1 // 32 + 40) * 8 * 4 * (4 + 64) * 256
    assert required < tb.attention_workspace_bytes(40, 1, 61440, 32, 8) >= 40 * 8 * 15 * 9216
    a, b = both(32, 8, lens_q, lens_k, causal, ws_bytes=required)
    assert torch.equal(a, b)
    with pytest.raises(tb.TbikError):
        both(32, 8, lens_q, lens_k, causal, ws_bytes=required - 256)


def test_oracle_parity():
    c = syn.attention_inputs(61, [1, 2, 1, 4], [4500, 70, 1000, 260], Hq=8, Hkv=2, D=128)
    Q, K, V = gu.dev_bf16(c["Q"]), gu.dev_bf16(c["K"]), gu.dev_bf16(c["V"])
    O = tb.tbik_attention(Q, K, V, i32(c["cu_q"]), i32(c["cu_k"]), 4, c["scale"], True)
    check_against_oracle(gu.host_bf16_bits(O), c, True, min_equal=0.98)


def same_values(a, b, dtype):
    """Same bits wherever a value is not NaN, NaN in the same places (the payload of a NaN is no part of the result)."""
    a, b = a.view(dtype), b.view(dtype)
    nan = torch.isnan(a)
    return torch.equal(nan, torch.isnan(b)) and torch.equal(a.view(torch.int16)[~nan], b.view(torch.int16)[~nan])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("value", [float("inf"), -float("inf"), float("nan")])
@pytest.mark.parametrize("where", ["last", "first", "last of K"])
def test_values_that_are_not_finite(dtype, value, where):
    """Tiles past the end of a sequence contribute nothing whatever its last key and value are: key counts that end on a tile
    edge inside a round of four tiles (64, 128, 192), on a round (256), inside a tile (65), behind a split (4160)."""
    lens = [64, 128, 192, 256, 65, 320, 4160]

    def poison(K, V, starts, ends):
        for i, (s, e) in enumerate(zip(starts, ends)):
            if where == "last of K":
                K[e - 1, i % 2, 5] = value
            else:
                V[e - 1 if where == "last" else s, i % 2, 3::7] = value
    for lens_q in ([1] * len(lens), [3] * len(lens)):
        a, b = both(8, 2, lens_q, lens, dtype=dtype, seed=3, edit=poison)
        assert same_values(a, b, dtype)
        if where == "last" and value == float("inf") and lens_q[0] == 1:          # inf and not 0 x inf where no tile is ragged
            assert torch.isinf(a.view(dtype)[:4]).any(dim=2).any(dim=1).all() and not torch.isnan(a.view(dtype)[:4]).any()


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("Hq,Hkv,said_q,lens_q", [(8, 2, 1, [3, 0, 1, 0, 0, 2]), (8, 2, 2, [3, 1]), (8, 2, 8, [17, 1, 0, 9]), (4, 4, 3, [8, 1, 0]),
                                                  (32, 1, 1, [2, 0, 1]), (8, 2, 5, [0, 21, 1, 1, 2, 0])])
def test_a_sequence_with_more_queries_than_max_seqlen_q(Hq, Hkv, said_q, lens_q, causal):
    """batch x max_seqlen_q covers the call's tokens, so every query is computed, whichever sequence it belongs to; keys of one
    tile, of several rounds and of two splits (whose states the first max_seqlen_q queries pass through the workspace)."""
    assert said_q * len(lens_q) >= sum(lens_q) and max(lens_q) > said_q
    for lens_k in ([4500] * len(lens_q), [70 + 200 * i for i in range(len(lens_q))], [5] * len(lens_q)):
        a, b = both(Hq, Hkv, lens_q, lens_k, causal, seed=said_q, said_q=said_q)
        assert torch.equal(a, b)


def test_more_workgroups_than_a_launch_of_this_kernel_holds():
    """65535 sequences (three of them with a query) on 128 heads: 8.4 million items of 768 threads are past the limit of 2^32
    threads, attention_kernel's are not."""
    lens_q, lens_k = [0] * 65532 + [1, 1, 1], [0] * 65532 + [100, 64, 300]
    a, b = both(128, 128, lens_q, lens_k)
    assert torch.equal(a, b) and not (b == torch.tensor(7.0, dtype=torch.bfloat16).view(torch.int16)).all(dim=2).any()


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("Hq,Hkv,q,batches,keys", [(64, 8, 4, (16, 17), 100), (64, 8, 4, (32, 33), 300), (32, 32, 1, (8, 9), 64), (16, 8, 1, (96, 97), 40),
                                                   (16, 16, 1, (16, 17, 18, 19), 1030), (16, 16, 2, (22, 23), 2100), (32, 8, 1, (32, 33, 40, 41), 3001)])
def test_both_sides_of_the_lines_between_the_two_kernels(Hq, Hkv, q, batches, keys, causal):
    """Sizes next to each line of the rule that gives a call of few queries to one kernel or the other: same bits on both sides, and
    for sequences of one length as for ragged ones, which the rule tells apart."""
    for B in batches:
        for lens_k in ([keys] * B, [keys - (i * 37) % (keys - 8) for i in range(B)]):
            a, b = both(Hq, Hkv, [q] * B, lens_k, causal, seed=B)
            assert torch.equal(a, b), (B, lens_k[-1])

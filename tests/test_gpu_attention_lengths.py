"""Decode attention whose chunks follow the lengths (several sequences in
long chunks): against the oracle at the edges of that split, and with the
sequences it must keep apart."""

from __future__ import annotations

import numpy as np
import pytest

import attn_cases
from gpu_util import announce
from test_gpu_attention import check_tolerance, gpu_attention

pytestmark = pytest.mark.gpu

# (query heads, kv heads, page, lengths, max_seq_len): the bound on the
# lengths makes the fixed chunks at least 512 tokens long.
CASES = [
    (24, 8, 16, (8192, 1, 0, 300, 257), 8192),           # one sequence holds nearly all chunks
    (32, 8, 16, (2048,) * 16, 2048 * 2),                 # equal lengths, a loose bound
    (7, 1, 32, tuple(range(0, 4200, 60)), 4200),         # 70 sequences: two per lane; one workgroup per CU
    (16, 2, 64, (1, 0, 0, 2, 0), 40000),                 # almost nothing to do under a loose bound
    (4, 4, 1, (700, 64, 65, 128, 8000), 8000),           # pages of one token
    (6, 2, 16, tuple(64 * i for i in range(1, 131)), 8320),  # 130 sequences of whole chunk quanta
    # Six query heads or more under a long bound: the block-table entries of the longest chunk have to fit the LDS.
    (28, 4, 1, tuple(1 + 13 * i for i in range(63)) + (20000,), 41000),
    (64, 8, 1, tuple(5 + 29 * i for i in range(31)) + (9000,), 65536),
    (48, 8, 16, tuple(3 + 70 * i for i in range(15)) + (17000,), 1 << 20),
]


@pytest.mark.parametrize("hq,hkv,page,lens,max_len", CASES, ids=[f"hq{c[0]}_hkv{c[1]}_S{len(c[3])}" for c in CASES])
def test_lengths_against_oracle(hq, hkv, page, lens, max_len, monkeypatch):
    announce(f"attention by length hq={hq} hkv={hkv} S={len(lens)} max={max_len}")
    case = attn_cases.random_case(300 + hq + len(lens), hq, hkv, 128, page, lens, extra_pages=3)
    got = gpu_attention(case, max_seq_len=max_len)
    check_tolerance(case, got, "by length")
    assert np.all(got[np.asarray(lens) == 0] == 0)
    # the same values within the tolerance as with chunks of one length
    monkeypatch.setenv("WQ_ATTN_BY_LENGTH", "0")
    check_tolerance(case, gpu_attention(case, max_seq_len=max_len), "fixed chunks")


def test_lengths_invalid_sequences_stay_apart():
    """A bad length or page makes that sequence's output NaN and leaves the
    others within the tolerance."""
    announce("attention by length, invalid sequences")
    lens = (5000, 90, 700, 80, 1500)
    case = attn_cases.random_case(71, 24, 8, 128, 16, lens, extra_pages=2, max_pages=600)
    table = case.block_table.copy()
    table[2, 40] = case.k_cache.shape[0]
    bad_lens = case.seq_lens.copy()
    bad_lens[1], bad_lens[3] = 8193, -1
    got = gpu_attention(case._replace(block_table=table, seq_lens=bad_lens), max_seq_len=8192)
    for s in (1, 2, 3):
        assert np.all(np.isnan(got[s].astype(np.float32))), s
    keep = [0, 4]
    check_tolerance(attn_cases.select_sequences(case, keep), got[keep], "valid sequences")


@pytest.mark.parametrize("hq,hkv", [(24, 8), (8, 1)])
def test_lengths_many_invalid_sequences(hq, hkv):
    """Two thirds of the sequences have a bad or an empty length, so their
    merges write at once, without a unit to read: NaN or zeros in every
    element, and the others within the tolerance."""
    lens = tuple(0 if i % 3 == 1 else 700 + 97 * i for i in range(48))
    announce(f"attention by length, many invalid sequences hq={hq}")
    case = attn_cases.random_case(72 + hq, hq, hkv, 128, 16, lens, extra_pages=2, max_pages=600)
    bad_lens = case.seq_lens.copy()
    bad = np.arange(len(lens)) % 3 == 2
    bad_lens[bad] = np.where(np.arange(bad.sum()) % 2, -1, 8193)
    got = gpu_attention(case._replace(seq_lens=bad_lens), max_seq_len=8192)
    assert np.all(np.isnan(got[bad].astype(np.float32)))
    assert np.all(got[np.asarray(lens) == 0] == 0)
    keep = [i for i in range(len(lens)) if i % 3 == 0]
    check_tolerance(attn_cases.select_sequences(case, keep), got[keep], "valid sequences")


def test_whole_short_sequences_need_no_workspace():
    """Up to 192 tokens one workgroup takes a sequence whole."""
    from paper_2412_15803_amd import wq

    for n in (65, 128, 192):
        assert wq.paged_attention_workspace_size(1, 24, 8, 128, n) == 0
        announce(f"attention whole sequence of {n}")
        case = attn_cases.random_case(500 + n, 24, 8, 128, 16, (n, n - 64), extra_pages=1)
        check_tolerance(case, gpu_attention(case), f"{n} tokens")
    assert wq.paged_attention_workspace_size(1, 24, 8, 128, 193) > 0

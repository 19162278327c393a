"""GPU parity of the high-frequency list builder (Sec. 2.2 corpus statistics) against the oracle: counts, the list and
the number of skipped ids, all bit-exact (integer work)."""
import numpy as np
import pytest

from paper_2509_18362_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available()
    from oracle import oracle as orc_mod
    from paper_2509_18362_amd import binding
    return {"torch": torch, "orc": orc_mod, "binding": binding}


def both(gpu, tokens, V, n):
    torch, binding = gpu["torch"], gpu["binding"]
    want = gpu["orc"].build_subset(tokens, V, n)
    dev = torch.from_numpy(np.ascontiguousarray(tokens, dtype=np.int32)).to("cuda:0")
    got = binding.build_subset(dev, V, n, want_counts=True)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got["counts"].cpu().numpy().astype(np.int64), want["counts"])
    assert int(got["invalid"].cpu().numpy()[0]) == want["invalid"]
    np.testing.assert_array_equal(got["ids"].cpu().numpy(), want["ids"])
    return want


def both_entry_points(gpu, tokens, V, n):
    """And the entry point without a workspace, as far as its vocabularies go."""
    torch, binding = gpu["torch"], gpu["binding"]
    want = both(gpu, tokens, V, n)
    if V > binding.mtp_subset_static_max_vocab():
        return
    dev = torch.from_numpy(np.ascontiguousarray(tokens, dtype=np.int32)).to("cuda:0")
    ids, counts, invalid = (torch.full((size,), -7, dtype=torch.int32, device="cuda:0") for size in (n, V, 4))
    torch.cuda.synchronize()
    assert binding.mtp_subset_build_static(dev, dev.numel(), V, n, ids, counts, invalid, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    np.testing.assert_array_equal(counts.cpu().numpy().astype(np.int64), want["counts"])
    assert int(invalid.cpu().numpy()[0]) == want["invalid"]
    np.testing.assert_array_equal(ids.cpu().numpy(), want["ids"])


@pytest.mark.parametrize("V,N,n", [(7, 40, 3), (16, 10, 12), (50, 2001, 50), (50, 2003, 0), (33, 500, 5), (5, 0, 2),
                                   (1, 9, 1), (300, 7, 299)])
def test_small_streams_with_ties_and_invalid_ids(gpu, V, N, n):
    """Tiny vocabularies: ties at the cut, ids that never occur, ids out of range, an empty stream, stream lengths
    that are not multiples of the 16-byte load, n = 0 and n = V."""
    rng = np.random.default_rng(V * 1000 + N)
    both(gpu, rng.integers(-2, V + 2, size=N), V, n)


def test_worked_example(gpu):
    ex = np.array([0, 0, 0, 1, 2, 2, 2, 4, 4])
    for n, ids in ((3, [0, 2, 4]), (2, [0, 2]), (4, [0, 1, 2, 4])):
        assert both(gpu, ex, 5, n)["ids"].tolist() == ids


@pytest.mark.parametrize("V,logN,n", [(4096, 18, 819), (40000, 20, 8000), (40001, 20, 13), (100000, 21, 25000)])
def test_long_tailed_streams(gpu, V, logN, n):
    """Vocabularies of exactly one counting chunk, one id more, and several chunks; out-of-range ids planted."""
    toks = synth.make_token_stream(V, (1 << logN) + 3, seed=V % 97, invalid_every=1001)
    both(gpu, toks, V, n)


def test_full_vocabulary_and_use_as_output_head_list(gpu):
    """The 7B vocabulary (151680 ids, one counting chunk) with the paper's list sizes; the built list is accepted
    as a compressed-head id list by mtp_draft_init (ascending, unique, in range)."""
    binding = gpu["binding"]
    V = synth.SEVEN_B.vocab_size
    toks = synth.make_token_stream(V, (1 << 23) + 1, seed=3)
    for n in (16384, 32768):
        want = both(gpu, toks, V, n)
    tiny = synth.WORKLOADS["c1_tiny"]
    tt = synth.make_token_stream(tiny.shape.vocab_size, 1 << 16, seed=4)
    lst = both(gpu, tt, tiny.shape.vocab_size, 1024)["ids"]
    eng = binding.DraftEngine(tiny.shape, synth.make_weights(tiny), [lst], 1, 192, 1)
    assert eng.subset_size(0) == 1024
    eng.close()


@pytest.mark.parametrize("V", [80768, 80769, 155392, 155393, 201920, 201921])
def test_every_field_width_and_chunk(gpu, V):
    """The largest vocabulary of each field width and of a chunk, and one id more: hot ids at both ends and in the middle of the
    words, a long tail, ids out of range."""
    rng = np.random.default_rng(V)
    hot = rng.choice([0, 1, 2, 3, 4, V // 2, V - 2, V - 1], size=1 << 18)
    toks = np.concatenate([hot, rng.integers(-3, V + 3, size=(1 << 20) + 5)])
    rng.shuffle(toks)
    both(gpu, toks, V, V // 7)


@pytest.mark.parametrize("V,base,ids,logN", [
    (4096, 0, 1, 21),          # one id: every add goes to one field, whose wraps carry into a neighbour that never occurs
    (4096, 8, 2, 24),          # 16-bit fields that wrap together, the second one carried into by the first
    (100000, 40, 8, 20),       # 8 bits: whole words full at a time, so that a carry runs through several fields
    (100000, 99996, 4, 20),    # the last word
    (160000, 155, 400, 23),    # 6 bits, more ids that wrap than the table has room for
    (100000, 1000, 4000, 24),  # 8 bits: a few wraps each
    (160001, 159996, 5, 20),   # the last word of the last id has one field in use
    (160000, 155, 100, 23),    # two chunks (there are no fields of 6 bits any more: 160000 ids are two chunks of 16)
    (400000, 1000, 1500, 25),  # three chunks; more ids that wrap than the table of wraps has room for
])
def test_fields_that_wrap(gpu, V, base, ids, logN):
    """A field narrower than its count: exact counts whatever the order of the adds."""
    rng = np.random.default_rng(V + ids)
    toks = base + rng.integers(0, ids, size=(1 << logN) + 1)
    both(gpu, toks, V, 3)
    if logN <= 21:  # and in runs: all lanes of a wave at one field
        both(gpu, np.sort(toks), V, 3)


@pytest.mark.parametrize("V,N,n", [(300, (1 << 24) + 64, 1), (300, 1 << 16, 16), (5000, 4095 * 16, 16), (70000, 1 << 20, 60000)])
def test_selection_in_one_to_three_digits(gpu, V, N, n):
    """The cut at counts of 25, 13, 12 and few bits: the digits follow from n_tokens / n; ids that occur more often than that
    all share the last bucket."""
    rng = np.random.default_rng(N % 1009)
    toks = np.concatenate([np.zeros(N // 2, dtype=np.int64), rng.integers(0, V, size=N - N // 2)])
    both(gpu, toks, V, n)


@pytest.mark.parametrize("V", [100000, 155393, 200001, 250000, 400000])
@pytest.mark.parametrize("kind", ["padded", "out of range", "before a chunk"])
def test_tokens_that_are_not_ids_of_the_chunk(gpu, V, kind):
    """Rows half of padding, other numbers out of range, and ids that are frequent and lie right before a chunk's first (of two or
    three chunks), in vocabularies of every field width, one chunk and several: none of them may end up in another id's count."""
    rng = np.random.default_rng(V)
    n = 1 << 22
    toks = rng.integers(0, V, size=n)
    if kind == "padded":
        toks.reshape(-1, 256)[:, 128:] = -1
    elif kind == "out of range":
        toks[rng.random(n) < 0.4] = -1
        toks[rng.random(n) < 0.3] = -5
        toks[rng.random(n) < 0.1] = V
    else:
        first = [c * (-(-V // parts // piece) * piece) for parts in (2, 3) for c in range(1, parts) for piece in (16, 20)]
        hot = rng.random(n) < 0.6
        toks[hot] = rng.choice(np.array(first) - 1, size=int(hot.sum()))
    both_entry_points(gpu, toks, V, V // 7)


@pytest.mark.parametrize("V,ids,logN", [(60000, 3, 23), (100000, 40, 23), (151680, 60, 23), (200001, 60, 23), (250000, 700, 26)])
def test_fields_that_wrap_without_a_workspace(gpu, V, ids, logN):
    """One copy of the counts, fields added one by one: as many ids side by side as scattered, one chunk and two, in the last case
    more of them than the table of wraps holds."""
    rng = np.random.default_rng(V + ids)
    n = (1 << logN) + 3
    some = np.concatenate([V // 3 + np.arange(ids), rng.choice(V, ids)])
    both_entry_points(gpu, rng.choice(some, n), V, min(V, 2 * ids + 5))

"""GPU parity where the split of the work over workgroups can go wrong: remainders of the item lists.

Bars as in test_gpu_parity (bf16 inputs, fp32 accumulation, bf16 output).
"""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_parity import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("Hkv", [1, 2, 4, 8, 3])
@pytest.mark.parametrize("P,E", [([40], [257]), ([0, 100, 7], [513, 1, 300]), ([64, 64], [300, 300]),
                                 ([64] * 9, [300] * 9), ([0] * 3, [1100] * 3)])
def test_items_dealt_out_over_the_xcds(H, Hkv, P, E):
    """Numbers of items that no number of XCDs divides, with several XCDs to a KV head and with one; equal
    requests in contiguous ranges and, where these would differ too much, dealt out."""
    w = W.make_uniform("items", 51, len(P), 3 * Hkv, Hkv, P, E)
    want = oracle.attention_of(w)
    for splits in (1, 3):
        _check(H.gpu_attention(w, num_splits=splits), want, f"Hkv={Hkv} P={P} E={E} splits={splits}")


@pytest.mark.parametrize("G,Hkv", [(4, 2), (8, 1), (1, 3), (4, 8)])
@pytest.mark.parametrize("P,E,without", [                 # without: the groups of heads that also run without scratch
    ([300, 40, 0, 1000], [1, 257, 16, 1], (1,)),          # decode-shaped requests next to a row tile and a bit
    ([6000, 10, 3000, 0, 64], [1, 300, 4, 700, 65], ()),  # several key ranges for some requests, one for others
    ([2000, 31, 32, 33, 0], [2, 1, 1, 1, 1], ()),         # blocks of 32 keys: remainders
    ([4096, 50, 0], [0, 513, 1], (1, 4, 8)),              # a request without new tokens
    ([190, 40, 7], [1, 59, 1], (1, 4, 8)),                # small: no key ranges at all, rows of some requests missing
    ([50, 300, 120, 77, 190] * 5, [1, 1, 1, 1, 60] * 5, (1, 4, 8)),   # one range each is faster than ranges of their own
    ([12000, 300, 500], [130, 130, 1], ()),               # one long request in many ranges
])
def test_batches_of_unequal_lengths(H, G, Hkv, P, E, without):
    import paper_2511_03475_amd as cp

    w = W.make_uniform("mixed", 52, len(P), G * Hkv, Hkv, P, E)
    want = oracle.attention_of(w)
    case = H.DeviceCase(w)
    _check(H.gpu_attention(w), want, f"G={G} Hkv={Hkv} P={P} E={E}")
    # without room for partial results a batch takes a plan that needs none, unless ranges of 8 key tiles would
    # have to do without them: those calls are refused
    st = cp.cp_extend_attention(case.q, case.k_new, case.v_new, case.kv_pages, case.block_table, case.prefix_lens,
                                case.extend_lens, case.out, None, case.shape, None, 0, check=False)
    assert st == (cp.CP_OK if G in without else cp.CP_ERR_WORKSPACE)
    if st == cp.CP_OK:
        _check(case.out_bits(), want, f"no workspace G={G} Hkv={Hkv} P={P} E={E}")


@pytest.mark.parametrize("P,E,Hq,Hkv,part,ok", [
    ([3000], [128], 8, 2, 0.75, True), ([3000], [128], 8, 2, 0.5, True), ([3000], [128], 8, 2, 0.25, False),
    ([1500] * 3, [40] * 3, 8, 2, 0.5, True), ([500] * 2, [600] * 2, 8, 2, 0.75, True),     # one number of ranges for all
    ([500] * 2, [600] * 2, 8, 2, 0.5, False),
    ([700, 1000, 1400, 900], [300, 1, 1, 300], 8, 2, 0.5, True),                           # unequal lengths
    ([782, 64], [1, 254], 64, 8, 0.75, True), ([782, 64], [1, 254], 64, 8, 0.1, True),
    ([12000, 300, 500], [130, 130, 1], 8, 2, 0.75, False),
    ([3763, 1178], [1, 47], 10, 2, 0.379, True),          # a split request by request, which takes less than the best plan
    ([9000], [9], 8, 2, 0.25, True), ([9000], [9], 8, 2, 0.1, False),                      # decode-shaped
])
def test_less_scratch_than_asked_for(H, P, E, Hq, Hkv, part, ok):
    """A part of cp_workspace_bytes: the call takes a plan that fits and leaves what lies behind alone, or is
    refused and leaves everything alone."""
    import torch

    import paper_2511_03475_amd as cp

    w = W.make_uniform("part", 62, len(P), Hq, Hkv, P, E)
    case = H.DeviceCase(w)
    size = int(case.ws_bytes * part) // 256 * 256
    assert 0 < size < case.ws_bytes
    space = torch.full((case.ws_bytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda:0")
    case.out.fill_(0x1234)
    st = cp.cp_extend_attention(case.q, case.k_new, case.v_new, case.kv_pages, case.block_table, case.prefix_lens,
                                case.extend_lens, case.out, torch.cuda.current_stream(), case.shape, space, size, check=False)
    assert st == (cp.CP_OK if ok else cp.CP_ERR_WORKSPACE)
    got = case.out_bits()
    assert (space[size if ok else 0:] == 0x5A).all()
    if ok:
        _check(got, oracle.attention_of(w), f"P={P} E={E} {part} of the scratch")
    else:
        assert (got == 0x1234).all()


@pytest.mark.parametrize("B,P,E,G,Hkv,ranges,tail", [
    (33, 1500, 70, 1, 8, 6, 1),       # one item more than the CUs of an XCD, three wavefronts of rows
    (17, 1000, 150, 2, 8, 5, 2),      # two tiles a request, the last one of 44 rows; requests in turn longest and shortest first
    (11, 1500, 250, 3, 8, 9, 1),      # G divides neither tile nor wavefront; the shortest tile of the last request
    (17, 489, 136, 2, 8, 4, 2),       # the merge of up to 4 ranges
    (19, 1539, 36, 8, 8, 4, 6),
    (3, 0, 5382, 1, 4, 2, 2),         # several XCDs to a KV head, their items dealt out: 2, 4 and 8
    (1, 1533, 1040, 16, 4, 9, 1),
    (3, 213, 5427, 2, 2, 3, 1),
    (2, 1958, 1119, 16, 2, 7, 12),
    (1, 143, 5707, 12, 1, 2, 12),
])
def test_the_last_round_alone_is_split(H, B, P, E, G, Hkv, ranges, tail):
    """Equal requests whose items do not fill the last round: only its row tiles are split and merged, `tail` of each
    KV head in `ranges` key ranges.  Against the oracle, and every row against the unsplit call, also in a buffer of
    exactly the size asked for."""
    import torch

    import paper_2511_03475_amd as cp

    w = W.make_uniform("tail", 71, B, G * Hkv, Hkv, [P] * B, [E] * B)
    case = H.DeviceCase(w)
    size = case.ws_bytes
    assert (cp.cp_num_splits(case.shape), size) == (ranges, tail * ranges * 256 * Hkv * 130 * 4)   # of its row tiles only
    case.workspace = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda:0")
    case.attention()
    got = case.out_bits()
    assert (case.workspace[size:] == 0x5A).all()
    _check(got, oracle.attention_of(w), f"tail B={B} P={P} E={E} G={G} Hkv={Hkv}")
    _check(H.gpu_attention(w, num_splits=1), W.bf16_bits_to_f32(got).astype(np.float64), "unsplit")


@pytest.mark.parametrize("P,E,G,Hkv,ranges,by_request", [
    ([0] * 3, [959] * 3, 4, 2, 1, False), ([70], [383], 3, 8, 1, False),       # equal requests
    ([2], [66], 16, 8, 1, False), ([0] * 3, [215] * 3, 3, 8, 1, False),        # ... 32 rows in the last tile, 5 in it
    ([1345] * 2, [58] * 2, 4, 1, 8, False), ([0], [1287], 1, 8, 3, False),     # ... in key ranges
    ([0, 130, 500], [900, 257, 1], 4, 2, 1, False), ([200, 0], [129, 1000], 2, 4, 1, False),       # unequal
    ([843, 285, 54, 0, 0], [66, 3, 229, 1, 436], 4, 1, 4, False),              # ... in one number of key ranges
    ([0, 1213, 36, 98, 7, 119], [1, 74, 87, 25, 406, 103], 4, 4, 6, True),     # ... split request by request
])
def test_row_tiles_of_half_the_rows(H, P, E, G, Hkv, ranges, by_request):
    """Calls whose row tiles do not fill the device, tiles of 128 rows: remainders, one row too many, splits."""
    import paper_2511_03475_amd as cp

    w = W.make_uniform("half", 72, len(P), G * Hkv, Hkv, P, E)
    case = H.DeviceCase(w)
    assert (cp.cp_plan_tile_rows(case.shape), cp.cp_num_splits(case.shape)) == (128, ranges)
    if ranges > 1:
        assert by_request == (case.ws_bytes < ranges * sum(E) * G * Hkv * 130 * 4)   # not every request in as many
    want = oracle.attention_of(w)
    _check(H.gpu_attention(w), want, f"half P={P} E={E} G={G} Hkv={Hkv}")
    _check(H.gpu_attention(w, num_splits=2), want, f"full P={P} E={E} G={G} Hkv={Hkv}")


@pytest.mark.parametrize("P", [1, 63, 65, 127, 129, 191, 449, 450])
def test_a_prefix_that_ends_inside_a_tile(H, P):
    """The steady-state loop runs over the prefix, is left for the tile the prefix ends in, and runs on over the
    new keys; ranges that begin and end around that tile too."""
    w = W.make_uniform("ragged", 73, 1, 2, 2, [P], [700])
    want = oracle.attention_of(w)
    for splits in (1, 2, 5):
        _check(H.gpu_attention(w, num_splits=splits), want, f"P={P} splits={splits}")


def test_more_requests_than_lanes(H):
    """70 requests of both kinds: two groups of 64 in every search, equal lengths among the sorted ones."""
    rng = np.random.default_rng(53)
    P = [int(x) for x in rng.integers(0, 700, 70)]
    E = [int(x) for x in np.where(rng.random(70) < 0.7, 1, rng.integers(20, 90, 70))]
    P[3] = P[66] = 2500
    P[5:9], E[5:9] = [128] * 4, [64] * 4
    w = W.make_uniform("mixed70", 53, 70, 8, 2, P, E)
    _check(H.gpu_attention(w), oracle.attention_of(w), "70 requests")


@pytest.mark.parametrize("P,E", [([512], [128]), ([0], [300]), ([130], [65]), ([900, 900], [33, 33]), ([64], [64]),
                                 ([3000], [128]), ([3000, 100], [100, 128])])
def test_short_key_ranges(H, P, E):
    """Few row tiles: a workgroup per 32 rows, or key ranges of a few tiles; then without room for partial
    results, where a short call does without and a longer one is refused."""
    import paper_2511_03475_amd as cp

    w = W.make_uniform("ranges", 54, len(P), 8, 2, P, E)
    want = oracle.attention_of(w)
    case = H.DeviceCase(w)
    _check(H.gpu_attention(w), want, f"P={P} E={E}")
    st = cp.cp_extend_attention(case.q, case.k_new, case.v_new, case.kv_pages, case.block_table, case.prefix_lens,
                                case.extend_lens, case.out, None, case.shape, None, 0, check=False)
    # 49 key tiles make six ranges of 8: too long to go without scratch
    assert st == (cp.CP_ERR_WORKSPACE if P[0] == 3000 else cp.CP_OK)
    if st == cp.CP_OK:
        _check(case.out_bits(), want, f"no workspace P={P} E={E}")


@pytest.mark.parametrize("Hkv", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("E", [[1], [3, 0, 2], [1] * 70 + [37], [16, 1, 64, 5]])
def test_cache_append_remainders(H, Hkv, E):
    """Rows in numbers that no wavefront (4 rows) or workgroup (16) divides, odd numbers of KV heads, owners
    in the second group of 64 requests: every byte of the pool as the oracle leaves it."""
    P = [(7 * r) % 45 for r in range(len(E))]
    w = W.make_uniform("append", 55, len(E), Hkv, Hkv, P, E)
    case = H.DeviceCase(w)
    case.write_kv()
    want = oracle.write_kv(w.k_new, w.v_new, w.kv_pages, w.block_table, w.prefix_lens, w.extend_lens)
    assert np.array_equal(case.kv_pages.cpu().numpy().view(np.uint16), want.view(np.uint16))


@pytest.mark.parametrize("G,Hkv", [(4, 2), (8, 1), (1, 3), (5, 1)])
@pytest.mark.parametrize("P,E", [
    ([3000, 5, 0, 700], [1, 3, 2, 1]),      # one block of 32 rows; several workgroups a request, some without keys
    ([9000], [9]), ([2500, 31], [12, 7]),   # two blocks of 32 rows, the second one partly or wholly padding
    ([300], [11]), ([0], [5]), ([31, 33], [8, 8]),    # and so few keys that each block is a workgroup
    ([100], [65]), ([200, 200], [40, 40]), ([0, 64], [97, 97]),   # small row-tiled calls: a head's rows across two blocks
])
def test_decode_shaped_and_small_calls(H, G, Hkv, P, E):
    w = W.make_uniform("few_rows", 56, len(P), G * Hkv, Hkv, P, E)
    _check(H.gpu_attention(w), oracle.attention_of(w), f"G={G} Hkv={Hkv} P={P} E={E}")


def test_small_call_lets_nan_through(H):
    """A key that is not a number reaches every row that sees it, whichever wavefront read it."""
    import torch

    w = W.make_uniform("nan", 57, 1, 8, 2, [300], [100])
    case = H.DeviceCase(w)
    page = int(case.block_table[0, 9])                    # tokens 144 .. 159
    case.kv_pages.view(-1)[(page * 2 * 2 + 1) * 16 * 128 + 5 * 128] = 0x7FC0      # K of KV head 1
    case.attention()
    out = case.out.view(torch.bfloat16).float()
    assert out[:, 4:].isnan().all() and not out[:, :4].isnan().any()


@pytest.mark.parametrize("splits", [8, 9, 16, 17, 32, 33])
@pytest.mark.parametrize("E", [31, 32])
def test_merge_forms(H, splits, E):
    """Both forms of the merge around the limits of their numbers of ranges, with 1024 (row, head) pairs and
    fewer; some ranges are empty."""
    w = W.make_uniform("merge", 58, 1, 32, 8, [1500], [E])
    _check(H.gpu_attention(w, num_splits=splits), oracle.attention_of(w), f"E={E} splits={splits}")


@pytest.mark.parametrize("P,E,splits", [
    ([3000, 6000, 10, 0], [130, 1, 300, 700], 0),         # a mixed batch: its own merge
    ([3000, 40], [1, 300], 0),                            # ... whose decode-shaped request is the bad one
    ([1500], [100], 3), ([1500], [100], 7),               # the merge of few ranges, at each of its sizes
    ([1500], [130], 12), ([1500], [130], 23),
    ([1500], [130], 40), ([1500], [9], 23),               # the merge of many
    ([3000], [1], 0), ([40000], [9], 0),                  # decode-shaped: LDS sum, then a merge
    ([1500], [130], 1),                                   # and none at all
])
def test_bad_keys_come_through_every_merge(H, P, E, splits):
    """A key or a value that is not a number makes every row that sees it not a number, also where another
    range of the row's keys outweighs it by far; so do scores that are all minus infinity (0 / 0, as in the
    oracle).  Heads of the other KV head stay finite."""
    import torch

    w = W.make_uniform("bad", 59, len(P), 8, 2, P, E)
    token = P[0] // 2
    page, rows = int(w.block_table[0, token // 16]), E[0]
    for what in (0, 1):                                   # K, V
        case = H.DeviceCase(w, splits)
        assert splits == 1 or case.ws_bytes > 0
        case.kv_pages.view(-1, 2, 2, 16, 128)[page, what, 1, token % 16, 5] = 0x7FC0
        case.attention()
        out = case.out.view(torch.bfloat16).float()
        bad = slice(None) if what == 0 else slice(5, 6)
        assert out[:rows, 4:, bad].isnan().all() and out[:, :4].isfinite().all(), f"what={what} P={P} E={E} splits={splits}"
    case = H.DeviceCase(w, splits)                        # key 3 outweighs all others, the bad value has weight 0
    pool = case.kv_pages.view(-1, 2, 2, 16, 128)
    case.q[:rows, 4:] = 0x4140                            # 12
    pool[int(w.block_table[0, 0]), 0, 1, 3] = 0x4140
    pool[page, 1, 1, token % 16, 5] = 0x7FC0
    case.attention()
    out = case.out.view(torch.bfloat16).float()
    assert out[:rows, 4:, 5].isnan().all() and out[:, :4].isfinite().all(), f"outweighed P={P} E={E} splits={splits}"
    case = H.DeviceCase(w, splits)
    case.q[:rows, 4:, 0] = 0x3F80                         # 1 times minus infinity
    case.kv_pages.view(-1, 2, 2, 16, 128)[:, 0, 1, :, 0] = -128        # 0xFF80
    case.k_new.view(-1, 2, 128)[:, 1, 0] = -128
    case.attention()
    out = case.out.view(torch.bfloat16).float()
    assert out[:rows, 4:].isnan().all() and out[:, :4].isfinite().all(), f"minus infinity P={P} E={E} splits={splits}"


@pytest.mark.parametrize("B,Hkv,P,E", [
    (7, 32, 1000, 9), (3, 3, 16000, 9),       # both blocks of rows in a wavefront; one workgroup on the keys, several
    (1, 2, 2513, 14), (3, 2, 1500, 11),       # apart, several workgroups: their number a multiple of the XCDs, and not
    (40, 8, 150, 13),                         # apart, one workgroup each
])
def test_two_blocks_of_rows_together_and_apart(H, B, Hkv, P, E):
    """Lengths that differ a little and requests without new tokens, so that blocks are partly or wholly padding."""
    Ps = [max(P - 37 * (r % 5), 0) for r in range(B)]
    Es = [E - r % 4 if r % 6 != 5 else 0 for r in range(B)]
    w = W.make_uniform("two_blocks", 60, B, 4 * Hkv, Hkv, Ps, Es)
    _check(H.gpu_attention(w), oracle.attention_of(w), f"B={B} Hkv={Hkv} P={P} E={E}")


@pytest.mark.parametrize("Hq,Hkv,P,E", [
    (8, 2, [1806, 191, 1026, 2831, 250, 6836, 113], [21, 21, 24, 23, 22, 26, 20]),     # split request by request
    (32, 8, [181, 99, 607, 1950, 821, 157, 4821, 6124], [1, 24, 23, 1, 1, 1, 1, 1]),
    (8, 2, [4000, 10, 3000], [130, 1, 300]), (32, 8, [10240], [128]),                  # one number of ranges for all
    (8, 2, [9000], [9]), (8, 2, [3000, 5, 0, 700], [1, 3, 2, 1]),                      # decode-shaped
])
def test_more_scratch_than_asked_for_changes_nothing(H, Hq, Hkv, P, E):
    """cp_workspace_bytes is what the best plan takes: with exactly that much the same plan is made as with any
    amount, bit for bit the same result."""
    import torch

    import paper_2511_03475_amd as cp

    w = W.make_uniform("room", 61, len(P), Hq, Hkv, P, E)
    case = H.DeviceCase(w)
    assert case.ws_bytes > 0
    case.attention()
    want = case.out_bits().copy()
    case.out.fill_(0x7FC1)
    space = torch.empty(256 << 20, dtype=torch.uint8, device="cuda:0")
    cp.cp_extend_attention(case.q, case.k_new, case.v_new, case.kv_pages, case.block_table, case.prefix_lens,
                           case.extend_lens, case.out, torch.cuda.current_stream(), case.shape, space, space.numel())
    assert (case.out_bits() == want).all()


@pytest.mark.parametrize("P,E,Hq,Hkv", [
    ([86, 2657, 810, 125, 3000], [1, 1, 167, 114, 1], 32, 8),      # row tiles of 14, 15 and 16 key tiles, 2 ranges
    ([5000, 0, 640, 12], [200, 1, 448, 1], 8, 2),                  # several ranges, more row tiles
    ([836, 0, 0, 0, 27, 0], [3, 75, 551, 195, 265, 216], 8, 4),    # tiles of 256 rows
])
def test_row_tiles_with_fewer_keys_than_their_requests_last(H, P, E, Hq, Hkv):
    """The ranges of a request split on its own: none longer than those of its last row tile, some of them empty."""
    import paper_2511_03475_amd as cp

    w = W.make_uniform("ranges", 71, len(P), Hq, Hkv, P, E)
    case = H.DeviceCase(w)
    ranges = cp.cp_num_splits(case.shape)
    assert ranges > 1 and 0 < case.ws_bytes < ranges * sum(E) * Hq * 130 * 4       # not every request in as many
    _check(H.gpu_attention(w), oracle.attention_of(w), f"P={P} E={E}")


@pytest.mark.parametrize("P,E,Hq,Hkv", [
    ([1500] * 33, [70] * 33, 8, 8),                        # equal requests, the last round split
    ([765, 885, 278, 30], [98, 337, 295, 347], 32, 8),     # split request by request
])
@pytest.mark.parametrize("off", [16, 128])
def test_a_misaligned_buffer_where_whole_head_tiles_asked_for_none(H, P, E, Hq, Hkv, off):
    """Row tiles of whole heads needed no scratch for these shapes, so a buffer that is not aligned was accepted
    and not looked at: the call runs as one without a buffer does, and leaves it alone."""
    import torch

    import paper_2511_03475_amd as cp

    case = H.DeviceCase(W.make_uniform("misaligned", 74, len(P), Hq, Hkv, P, E))
    assert case.ws_bytes > 0
    run = lambda space, size: cp.cp_extend_attention(case.q, case.k_new, case.v_new, case.kv_pages, case.block_table,  # noqa: E731
                                                     case.prefix_lens, case.extend_lens, case.out,
                                                     torch.cuda.current_stream(), case.shape, space, size)
    run(None, 0)
    want = case.out_bits().copy()
    case.out.fill_(0x1234)
    space = torch.full((case.ws_bytes + 512,), 0x5A, dtype=torch.uint8, device="cuda:0")
    run(space[off:], case.ws_bytes)
    assert (case.out_bits() == want).all() and (space == 0x5A).all()

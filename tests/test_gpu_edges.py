"""Edges of the kernels' tiles and of their dispatch rules, against the same oracles and rules as the other GPU tests."""
import numpy as np
import pytest
import torch

import oracle as O
import synth_inputs as syn
import test_gpu_parity as P
import test_placement_search as Q
from helpers import sample_rows
from paper_2401_08383_amd import binding as B

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[case] {msg}", flush=True)


# ----------------------------------------------------------------------------- trace columns of any length
@pytest.mark.parametrize("N", [3, 4, 5, 6, 7, 4097, 8190, 61441, 61443, 65537, 262145, 262147])
def test_trace_columns_that_start_and_end_anywhere(oracle, N):
    """Columns off the 16-byte grid, last vectors cut by one to three ids, last chunks shorter than a vector."""
    P.test_affinity_and_locality_parity(oracle, 5, N, 24, 8)
    Q.test_affinity_multihop_parity(4, N, 24)
    Q.test_routing_transfers_parity(5, N, 24, 8)


@pytest.mark.parametrize("L,N,E,G", [
    (2, 4, 1, 1), (3, 5, 64, 8), (2, 4095, 63, 7), (24, 4097, 64, 8), (2, 8191, 64, 8), (2, 8193, 8, 4), (5, 24575, 40, 5), (5, 24576, 2, 2), (5, 24577, 8, 4),
    (4, 11392, 8, 4), (4, 11393, 8, 4), (12, 10240, 8, 4), (12, 10241, 16, 4), (33, 16385, 3, 3), (33, 2000, 24, 4),
    (5, 24577, 64, 8), (24, 5120, 64, 8), (24, 5121, 64, 8), (24, 61443, 64, 8)])
def test_short_traces(oracle, L, N, E, G):
    """One launch a call up to a number of tokens that depends on the call, two beyond: both sides of it, tokens cut by the end of a sweep,
    invalid ids, few bins and as many as there are."""
    P.test_affinity_and_locality_parity(oracle, L, N, E, G)
    trace, _ = syn.planted_trace(L, N, E, 0.5, seed=2100 + N)
    g = syn.rng(2101 + L)
    bad = g.random((L, N)) < 0.02
    bad[L - 1, N - 1] = bad[0, 0] = True
    trace[bad] = g.choice(np.array([-1, E, 1 << 20, -(1 << 31)]), size=int(bad.sum())).astype(np.int32)
    P._affinity_case(oracle, trace, E, syn.balanced_random_placement(L, E, G, seed=2102), G)
    Q.test_affinity_multihop_parity(L, N, E)
    Q.test_routing_transfers_parity(L, N, E, G)


# chunks of whole wavefronts past one sweep, the last one cut; rows of 23, 31 and 32 words and an odd number of experts (words of two rows),
# groups of three pairs and of fewer
@pytest.mark.parametrize("L,N,E,G", [(24, 135001, 64, 8), (4, 40000, 62, 2), (23, 200003, 46, 2), (5, 300002, 64, 4), (24, 140001, 63, 7), (24, 131072, 44, 4),
                                     # partials of 7, 22 and (28 layer groups, one of them of a chunk an XCD) 8 chunks
                                     (22, 26562, 64, 4), (6, 90001, 40, 4), (85, 70000, 16, 4),
                                     # chunks of two sweeps for a round trip fewer, and one token more than they would do for; 34, 48 and 128 partials in equal trips
                                     (16, 239003, 64, 8), (16, 262145, 48, 8), (2, 139001, 24, 8), (7, 1000003, 8, 4)])
def test_locality_from_the_histograms_of_a_chunk(oracle, L, N, E, G):
    _say(f"statistics L={L} N={N} E={E} G={G}")
    trace, _ = syn.planted_trace(L, N, E, 0.5, seed=2150 + N)
    g = syn.rng(2151 + L)
    bad = g.random((L, N)) < 0.001
    bad[L - 1, N - 1] = bad[0, 0] = True
    trace[bad] = g.choice(np.array([-1, E, 1 << 20, -(1 << 31)]), size=int(bad.sum())).astype(np.int32)
    P._affinity_case(oracle, trace, E, syn.balanced_random_placement(L, E, G, seed=2152), G)


@pytest.mark.parametrize("N", [300, 262147, 414593])
def test_placement_of_all_layers_beyond_64_KiB(oracle, N):
    """The most layers and experts.  Up to 412992 tokens (locality 414592) a workgroup takes a layer and two rows of the placement; beyond,
    the placement of all layers and the counts take more LDS than a launch may use unasked.  Both calls twice: the second one relies
    on what the first has asked for."""
    for _ in range(2):
        Q.test_routing_transfers_parity(256, N, 64, 8)
    _say(f"placement_locality L=256 N={N}")
    g = syn.rng(1150)
    trace = g.integers(0, 64, size=(256, N)).astype(np.int32)
    pl = syn.balanced_random_placement(256, 64, 8, 1151)
    for _ in range(2):
        got = B.placement_locality(torch.from_numpy(trace).cuda(), torch.from_numpy(pl).cuda(), 8).cpu().numpy()
        np.testing.assert_array_equal(got, oracle.placement_locality(trace, pl))


# ----------------------------------------------------------------------------- counts of all layer pairs
@pytest.mark.parametrize("L,N,E", [(2, 65281, 64), (4, 5, 1), (5, 4100, 63), (8, 8193, 2), (9, 65280, 33), (12, 130561, 5), (13, 20000, 64), (16, 16385, 64),
                                   (17, 9000, 31), (29, 24577, 7), (31, 3, 64), (33, 12289, 64),
                                   (29, 49153, 7), (30, 90115, 33), (33, 16385, 64), (47, 20001, 16)])
def test_multihop_blocks(L, N, E):
    """Whole and cut blocks of layers, few and many of them, rows of odd length, chunks at the counters' limit."""
    Q.test_affinity_multihop_parity(L, N, E)


@pytest.mark.parametrize("L,N", [(1, 8192), (1, 8193), (2, 8193), (3, 8192), (3, 8193), (3, 9792), (3, 9793), (4, 9792), (4, 9793), (24, 41792), (24, 41793), (24, 43392), (24, 43393)])
def test_transfers_either_side_of_one_launch(oracle, L, N):
    Q.test_routing_transfers_parity(L, N, 8, 4)
    P.test_affinity_and_locality_parity(oracle, L, N, 8, 4)


# the last trace in one launch and the first in chunks, for each range of layers and experts
@pytest.mark.parametrize("L,N,E", [(2, 32768, 63), (11, 32769, 5), (12, 81920, 40), (15, 81921, 41), (13, 49152, 39), (14, 49153, 8), (16, 106496, 16), (23, 106497, 7),
                                   (24, 49152, 23), (26, 49153, 2), (25, 90112, 24), (32, 90113, 39), (24, 131072, 40), (27, 131073, 64), (33, 16384, 1), (34, 16385, 9),
                                   (58, 2047, 10), (58, 2047, 9), (58, 2048, 7), (58, 2048, 6), (100, 2048, 37), (101, 2048, 64)])
def test_multihop_either_side_of_one_launch(L, N, E):
    Q.test_affinity_multihop_parity(L, N, E)


@pytest.mark.parametrize("L,N,E", [(5, 1100003, 3), (8, 430001, 5), (12, 250000, 2), (13, 200003, 9), (16, 250001, 64)])
def test_multihop_blocks_of_few_layers(L, N, E):
    """Traces of few layers that are long enough for the blocks."""
    Q.test_affinity_multihop_parity(L, N, E)


@pytest.mark.parametrize("L,N,E", [(2, 1, 64), (2, 3, 1), (3, 4099, 63), (4, 61441, 33), (5, 7, 64), (7, 8195, 2), (11, 40001, 17), (17, 60003, 40),
                                   (18, 4096, 64), (19, 30001, 5), (22, 4097, 64)])
def test_multihop_groups(L, N, E):
    """One to three targets in the last group of a layer, columns that start anywhere, every number of replicas."""
    Q.test_affinity_multihop_parity(L, N, E)


def test_multihop_groups_fill_a_counter():
    """Every transition of the longest chunk in one 16-bit counter."""
    N = 61440 * 256 - 5
    _say(f"multihop L=2 N={N}, one transition only")
    trace = torch.full((2, N), 63, dtype=torch.int32, device="cuda")
    counts = B.affinity_multihop(trace, 64)["counts"]
    assert counts[0, 63, 63].item() == N and counts.sum().item() == N


# ----------------------------------------------------------------------------- candidate scores
@pytest.mark.parametrize("E,Bn,total", [(1, 1, 5), (33, 9, (1 << 31) - 1), (33, 9, 1 << 31), (64, 300, (1 << 31) - 1), (64, 300, 1 << 33),
                                        (63, 4099, 100000)])
def test_candidate_scores_around_the_32_bit_table(E, Bn, total):
    """Pair totals on both sides of the limit of the 32-bit table, parts of any sign and size, one part for all experts."""
    _say(f"placement_locality_from_counts E={E} B={Bn} total={total}")
    L = 3
    g = syn.rng(1200 + E + Bn)
    counts = np.zeros((L - 1, E, E), dtype=np.int64)
    for l in range(L - 1):
        cell = total // (E * E)
        counts[l] = cell
        counts[l, g.integers(0, E), g.integers(0, E)] += total - cell * E * E
        assert counts[l].sum() == total
    maps = g.choice(np.array([0, 1, 5, 1 << 20, -1, -(1 << 31)], dtype=np.int64), size=(Bn, L, E)).astype(np.int32)
    maps[0] = 7
    got = B.placement_locality_from_counts(torch.from_numpy(counts).cuda(), torch.from_numpy(maps).cuda()).cpu().numpy()
    assert got[0].tolist() == [total] * (L - 1)
    for b in range(0, Bn, max(1, Bn // 100)):
        np.testing.assert_array_equal(got[b], O.placement_locality_from_counts(counts, maps[b]))


# ----------------------------------------------------------------------------- streamed weights (few rows per expert, fp32)
@pytest.mark.parametrize("d,f", [(64, 64), (128, 576), (832, 320), (64, 4096)])
@pytest.mark.parametrize("counts", [[0, 1, 8, 9, 16, 17, 0, 31], [32, 33, 0, 64, 65, 7, 1, 3], [0, 0, 0, 1], [1], [100, 0, 0, 2, 0, 5]])
def test_streamed_ffn_row_tiles(oracle, counts, d, f):
    """Row tiles of every height, reductions shorter than the wavefronts share, blocks of every width."""
    P._ffn_case(oracle, "bf16", counts, d, f, 0, True, seed=1300 + d + f)


@pytest.mark.parametrize("counts,d,f", [
    ([200, 62, 35, 33, 17, 16, 9, 8, 7, 1, 0, 0, 0, 0, 0, 3], 64, 4160),   # blocks of 64 columns
    ([90, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1], 320, 8256),                    # 64, then 16
    ([3, 0, 33, 1, 0, 17, 33, 1, 1, 100, 65], 576, 1664)])                 # 32 in both contractions
def test_streamed_ffn_ranges_of_equal_cost(oracle, counts, d, f):
    """Rows so uneven that the workgroups' ranges are cut by cost: every block of every tile, for every block width."""
    P._ffn_case(oracle, "bf16", counts, d, f, 0, True, seed=1350 + d)


@pytest.mark.parametrize("T,d,f,E,k", [(1, 256, 1024, 8, 1), (3, 64, 64, 2, 2), (256, 192, 448, 1, 1), (257, 192, 448, 1, 1), (84, 128, 704, 3, 1), (90, 128, 704, 64, 2)])
def test_streamed_ffn_fused(oracle, T, d, f, E, k):
    """Gathered rows, scattered and scaled results, tokens without a resident expert; 256 and 257 rows are the two sides
    of the rule that selects the path."""
    P._fused_case(oracle, T, d, f, E, E, k, 1, True, seed=1400 + T)
    P._fused_case(oracle, T, d, f, E, max(1, E // 3), k, 0, False, seed=1401 + T)


@pytest.mark.parametrize("A", [32, 33, 64, 65, 128, 129])
def test_single_expert_on_both_sides_of_the_streaming_rule(oracle, A):
    """One expert whose rows fill 32, 64 or 128 of a row tile: 512 x 2112 streams all of them, 1536 x 3072 up to 64 rows."""
    P._ffn_case(oracle, "bf16", [A], 512, 2112, 0, True, seed=1360 + A)
    P._ffn_case(oracle, "bf16", [A], 1536, 3072, 0, False, seed=1361 + A)


# ----------------------------------------------------------------------------- grouped contraction (many rows per expert)
@pytest.mark.parametrize("d,f", [(64, 64), (128, 320), (192, 448), (320, 256), (576, 832)])
@pytest.mark.parametrize("counts", [[128, 129, 0, 192, 193], [64, 65, 1, 255, 256, 257], [287, 288, 289, 320, 321], [511, 544, 545, 576, 577], [0, 2049]])
def test_grouped_ffn_row_tiles(oracle, counts, d, f):
    """Tiles of every height and both widths, whole and cut ones, reductions from one K tile on."""
    P._ffn_case(oracle, "bf16", counts, d, f, 0, True, seed=1700 + d + f)


@pytest.mark.parametrize("counts,d,f", [([65, 128, 0, 64, 127], 320, 1088), ([100], 128, 4160), ([66, 129, 300, 96], 64, 576),
                                        ([100] * 13, 192, 1088), ([128, 65] * 9 + [1, 260], 128, 1024)])
def test_grouped_ffn_tiles_of_128_rows(oracle, counts, d, f):
    """Experts of 65 to 128 rows: a tile in pieces of 64 rows in launches of few tiles, whole in larger ones (the last two)."""
    P._ffn_case(oracle, "bf16", counts, d, f, 1, True, seed=1750 + d)


@pytest.mark.parametrize("d,f", [(64, 192), (128, 320), (576, 1024), (1088, 1984)])
@pytest.mark.parametrize("counts", [[129, 160, 192, 193, 256, 257, 288], [289, 320, 385, 65, 66], [128, 96, 97, 64, 33, 1, 260, 130, 577]])
def test_grouped_ffn_cut_tiles(oracle, counts, d, f):
    """Tiles of every height in eight, four and two pieces (64 x 192 to 1088 x 1984), across rows, columns and both."""
    P._ffn_case(oracle, "bf16", counts, d, f, 0, True, seed=1770 + d)


@pytest.mark.parametrize("counts,d,f", [([192, 193, 224, 225, 200] * 3, 64, 3328), ([193, 224, 223, 210] * 4, 1664, 64), ([385, 448, 447, 449, 193] * 4 + [200], 4096, 64),
                                        ([129, 160, 159, 140, 100] * 3, 64, 3328), ([129, 160, 161, 130] * 5, 64, 3392), ([129, 160, 131, 150] * 4, 1664, 64),
                                        ([161, 192, 129, 224] * 4, 64, 2624), ([289, 320, 310, 129, 160] * 4 + [2208], 4096, 64)])
def test_grouped_ffn_tiles_between(oracle, counts, d, f):
    """Whole tiles between 128 and 192, 192 and 256 rows: in the first contraction, in the second one of 128 columns and of 256, one and two to an
    expert; with taller ones in the launch, of one round and of more."""
    P._ffn_case(oracle, "bf16", counts, d, f, 0, True, seed=1790 + f)


@pytest.mark.parametrize("counts", [[4096, 4096], [4095, 0, 200, 4097], [4096, 4100, 300]])
def test_grouped_ffn_around_two_rounds(oracle, counts):
    """512 tiles of the first contraction and a few more: hidden rows written through, by some experts only, by none."""
    P._ffn_case(oracle, "bf16", counts, 64, 4096, 0, True, seed=1790)


# the least weights that are streamed: whole and cut tiles of every height that one workgroup reads, experts of several tiles and of none beside
# them, short and long reductions (16 and 128 K tiles, the column tiles of an XCD begin at different ones)
@pytest.mark.parametrize("counts,d,f", [
    ([1, 63, 64, 65, 96, 97, 128, 129, 160, 192, 193, 255, 256, 257, 288, 289, 700, 0] + [30] * 46, 1024, 1024),
    ([40, 0, 64, 65, 128, 129, 192, 193, 256, 300, 513, 33, 1, 0, 70, 90], 512, 8192), ([70, 33, 250, 140], 2048, 8192)])
def test_grouped_ffn_streamed_weights(oracle, counts, d, f):
    offsets = np.concatenate([[0], np.cumsum(counts)])
    P._ffn_case(oracle, "bf16", counts, d, f, 0, False, seed=1795, rows=sample_rows(offsets, 1, 1796))


@pytest.mark.parametrize("counts,d,f,act,bias", [
    ([1, 64, 65, 128, 160, 193, 224, 256, 257, 288, 700, 0] + [30] * 52, 1024, 1024, 1, True), ([70, 33, 250, 140], 2048, 8192, 1, False), ([129, 33, 300, 192], 2048, 8192, 0, True)])
def test_grouped_ffn_streamed_weights_of_either_activation(oracle, counts, d, f, act, bias):
    """The tanh form, and biases with either, in the instances that stream."""
    _say(f"streamed weights {len(counts)} experts {d} x {f} act={act} bias={bias}")
    offsets = np.concatenate([[0], np.cumsum(counts)])
    P._ffn_case(oracle, "bf16", counts, d, f, act, bias, seed=1797 + act, rows=sample_rows(offsets, 1, 1798))


@pytest.mark.parametrize("T,k,E,E_local,routing", [(3000, 1, 64, 64, "gate"), (2500, 2, 64, 64, "ids"), (33000, 1, 64, 64, "gate")])
def test_streamed_weights_of_a_layer(T, k, E, E_local, routing):
    """The layer and its calls, fused and not; 256 columns a tile in the second contraction (the last)."""
    _layer_against_calls(T, k, E, E_local, "bf16", True, routing, 1024, 1024)
    _layer_against_calls(T, k, E, E_local, "bf16", False, routing, 1024, 1024, ("x_sorted", "y_sorted"))


@pytest.mark.parametrize("T,d,f,E,k", [(700, 64, 192, 3, 1), (1500, 192, 320, 5, 2), (900, 320, 1088, 2, 2)])
def test_grouped_ffn_fused(oracle, T, d, f, E, k):
    P._fused_case(oracle, T, d, f, E, E, k, 1, True, seed=1800 + T)
    P._fused_case(oracle, T, d, f, E, max(1, E // 2), k, 0, False, seed=1801 + T)


@pytest.mark.parametrize("d,f", [(4, 4), (36, 20), (132, 260), (1028, 64)])
@pytest.mark.parametrize("counts", [[0, 1, 15, 16, 17, 64, 65], [300, 0, 5], [1]])
def test_exact_ffn_ragged(oracle, counts, d, f):
    P._ffn_case(oracle, "f32", counts, d, f, 0, True, seed=1500 + d + f)


# Every fp32 kernel forms the same partial sums: the rows of an expert come out the same in a list of any length, alone as in the company of other experts.
# Lists of one launch, of two in 16 and in 64 rows, reductions of one wavefront, two and four; fewer units of 32 than parts, a cut last one.
@pytest.mark.parametrize("d,f", [(4, 64), (36, 100), (96, 1096), (132, 1028), (256, 512), (512, 512), (64, 4096)])
def test_exact_rows_do_not_depend_on_the_list(d, f):
    _say(f"fp32 rows alone and in company {d} x {f}")
    g = torch.Generator(device="cuda")
    g.manual_seed(1560 + d + f)
    counts = [4000, 0, 3, 1997, 2001]
    A, E = sum(counts), len(counts)
    x = torch.randn((A, d), device="cuda", generator=g)
    w1, w2 = torch.randn((E, f, d), device="cuda", generator=g), torch.randn((E, d, f), device="cuda", generator=g)
    begin = [sum(counts[:e]) for e in range(E + 1)]
    y = B.moe_expert_ffn(x, torch.tensor(begin, dtype=torch.int32, device="cuda"), w1, w2)
    for e, n in [(0, 1), (0, 17), (0, 300), (0, 1500), (0, 4000), (2, 3), (3, 1997), (4, 65)]:
        mine = slice(begin[e], begin[e] + n)
        alone = B.moe_expert_ffn(x[mine].contiguous(), torch.tensor([0, n], dtype=torch.int32, device="cuda"), w1[e:e + 1], w2[e:e + 1])
        assert torch.equal(alone, y[mine]), (e, n)


# both contractions by one workgroup a row tile: last columns and reductions of any length, tiles of one row, experts without rows, either side
# of the line (a long list of few tiles, weights that do not fit, the last list that a first contraction sorts)
@pytest.mark.parametrize("d,f", [(4, 4), (36, 20), (132, 260), (256, 1024), (68, 2052)])
@pytest.mark.parametrize("counts", [[0, 1, 1500, 16, 17, 64, 65], [3001, 0, 5], [1025], [1024], [160] * 16])
@pytest.mark.parametrize("act", [0, 1])
def test_exact_ffn_in_one_launch(oracle, counts, d, f, act):
    P._ffn_case(oracle, "f32", counts, d, f, act, act == 0, seed=1540 + d + f)


# gather, scale, scatter and clearing of that kernel against the oracle: tiles of one row, experts without rows, half of the experts elsewhere, none of the
# tokens here, two assignments a token
@pytest.mark.parametrize("T,E,E_local,k,d,f,skew", [
    (3001, 9, 9, 1, 44, 212, True), (3001, 9, 4, 1, 256, 92, False), (2000, 5, 5, 2, 96, 132, False), (1100, 64, 32, 1, 28, 52, False), (1100, 16, 7, 2, 60, 100, True)])
def test_exact_fused_layer_in_one_launch_parity(oracle, T, E, E_local, k, d, f, skew):
    _say(f"fused fp32 layer against the oracle T={T} E={E} E_local={E_local} k={k} {d} x {f}")
    P._fused_case(oracle, T, d, f, E, E_local, k, k - 1, E_local < E, seed=1570 + T + d, skew=skew, dtype="f32")


def test_exact_fused_layer_in_one_launch_without_rows():
    """Every expert lives elsewhere: nothing but zeros."""
    g = torch.Generator(device="cuda")
    g.manual_seed(1580)
    x = torch.randn((2000, 44), device="cuda", generator=g)
    w1, w2 = torch.randn((3, 212, 44), device="cuda", generator=g), torch.randn((3, 44, 212), device="cuda", generator=g)
    maps = B.moe_dispatch(x, torch.full((2000, 1), 5, dtype=torch.int32, device="cuda"), 6, E_local=3, gather=False)
    out = torch.full_like(x, -7)
    B.moe_expert_ffn_fused(x, maps.src_of_sorted, maps.sorted_of_src, torch.ones((2000, 1), device="cuda"), maps.expert_offsets, w1, w2, out=out)
    assert torch.equal(out, torch.zeros_like(out))


@pytest.mark.parametrize("T,k,E,E_local,fused,routing,d,f", [
    (3001, 1, 9, 9, True, "gate", 44, 212), (3001, 1, 9, 4, True, "ids", 256, 92), (2000, 2, 5, 5, True, "gate", 96, 132), (5000, 1, 3, 1, True, "dropped", 32, 128),
    (3001, 1, 9, 4, False, "ids", 100, 60), (1100, 2, 16, 16, False, "gate", 64, 128), (4096, 1, 16, 16, False, "gate", 256, 1024)])
def test_exact_layer_in_one_launch(T, k, E, E_local, fused, routing, d, f):
    _say(f"fp32 layer T={T} k={k} E={E} E_local={E_local} fused={fused} {routing} {d} x {f}")
    _layer_against_calls(T, k, E, E_local, "f32", fused, routing, d, f, () if fused else ("x_sorted", "y_sorted"))


# lists that are sorted by the one launch: the longest, tiles of one row and of 16, invalid ids and tokens without an expert here, also all of them
@pytest.mark.parametrize("T,k,E,E_local,fused,routing,d,f", [
    (1024, 1, 8, 8, True, "gate", 64, 256), (1023, 1, 64, 64, True, "ids", 4, 4), (1000, 1, 9, 4, True, "ids", 36, 20), (512, 1, 1, 1, True, "gate", 32, 128),
    (700, 1, 14, 14, False, "ids", 44, 300), (1024, 1, 9, 9, True, "dropped", 60, 64), (512, 2, 8, 8, False, "gate", 64, 256), (500, 2, 7, 3, False, "ids", 12, 68),
    # rows of several wavefronts' width that are cleared; a share of the experts
    (900, 1, 29, 29, True, "ids", 468, 564), (1024, 1, 29, 29, False, "dropped", 468, 564), (1000, 1, 16, 2, True, "ids", 64, 256), (999, 1, 16, 1, False, "gate", 64, 256),
    (900, 1, 58, 29, True, "ids", 468, 564)])
def test_exact_layer_that_sorts_in_one_launch(T, k, E, E_local, fused, routing, d, f):
    _say(f"fp32 layer T={T} k={k} E={E} E_local={E_local} fused={fused} {routing} {d} x {f}")
    _layer_against_calls(T, k, E, E_local, "f32", fused, routing, d, f, () if fused else ("x_sorted", "y_sorted"))


def test_exact_ffn_in_place():
    """Rows that are written where they were read: the same results in two launches."""
    g = torch.Generator(device="cuda")
    g.manual_seed(1590)
    x = torch.randn((3000, 64), device="cuda", generator=g)
    w1, w2 = torch.randn((5, 128, 64), device="cuda", generator=g), torch.randn((5, 64, 128), device="cuda", generator=g)
    off = torch.tensor([0, 700, 700, 1500, 2999, 3000], dtype=torch.int32, device="cuda")
    y = B.moe_expert_ffn(x, off, w1, w2)
    ws = torch.empty(B.lib().moe_expert_ffn_workspace_bytes(3000, 64, 128, 5, B.EXF_F32), dtype=torch.uint8, device="cuda")
    B._check(B.lib().moe_expert_ffn(x.data_ptr(), off.data_ptr(), w1.data_ptr(), None, w2.data_ptr(), None, 3000, 64, 128, 5, 0, B.EXF_F32, x.data_ptr(),
                                    ws.data_ptr(), ws.numel(), B._stream()))
    assert float((x - y).abs().max()) <= 1e-5 * float(y.abs().max())


@pytest.mark.parametrize("T,k,over", [(512, 1, ["out"]), (1024, 1, ["out"]), (1024, 1, ["y_sorted"]), (700, 1, ["out", 4096]), (512, 2, ["y_sorted"]), (512, 2, ["y_sorted", 4096])])
def test_exact_layer_over_the_sorted_copies(T, k, over):
    """Results in the buffer of the sorted copies, which are dead by then, or reaching into it: those of the calls, which write them in launches of their own."""
    from paper_2401_08383_amd.pipeline import MoELayerRun

    _say(f"fp32 layer, T={T} k={k}, {over} over the sorted copies")
    g = torch.Generator(device="cuda")
    g.manual_seed(1595 + T)
    x, wg, w1, w2 = (torch.randn(shape, device="cuda", generator=g) for shape in ((T, 64), (8, 64), (8, 256, 64), (8, 64, 256)))
    idx = torch.randint(-1, 9, (T, k), device="cuda", generator=g, dtype=torch.int32)
    run = MoELayerRun(x, wg, w1, w2, k, k > 1, topk_idx=idx)
    run.step()
    ref = run.out.clone()
    room = torch.zeros(T * k * 64 + 4096, device="cuda")
    run.x_sorted = room[:T * k * 64].view(T * k, 64)
    begin = sum(over[1:])  # floats
    setattr(run, over[0], room[begin:begin + T * k * 64].view(T * k, 64))
    for _ in range(3):
        room.fill_(-7)
        run.step()
        assert torch.equal(run.out, ref)


# ----------------------------------------------------------------------------- dispatch: every workgroup counts the whole list
@pytest.mark.parametrize("T,k,d,E,E_local", [
    (1, 1, 8, 1, 1), (7, 1, 72, 3, 3), (9, 2, 1032, 64, 64), (2048, 2, 64, 8, 8), (4097, 1, 136, 40, 7), (3584, 2, 16, 64, 64), (7169, 1, 16, 64, 64),
    (6144, 1, 376, 9, 9), (6145, 1, 376, 9, 9), (7168, 1, 384, 2, 2), (7169, 1, 384, 2, 2)])
def test_dispatch_rows_in_one_launch(oracle, T, k, d, E, E_local):
    """Slices of 8 and of 16 assignments, cut by the end of the list, ragged rows, dropped assignments; the first size past them, for
    short rows and for others."""
    _say(f"dispatch rows T={T} k={k} d={d} E={E} E_local={E_local}")
    g = syn.rng(2000 + T)
    x = syn.quantize(g.standard_normal((T, d), dtype=np.float32), "bf16")
    idx = g.integers(-1, E + 1, size=(T, k)).astype(np.int32)
    expert_map = None
    if E_local < E:
        expert_map = np.full(E, -1, dtype=np.int32)
        expert_map[g.permutation(E)[:E_local]] = np.arange(E_local, dtype=np.int32)
    P._run_dispatch(oracle, x, idx, E, E_local, expert_map, "bf16")


@pytest.mark.parametrize("A,E,E_local", [(1, 1, 1), (255, 64, 64), (257, 2, 2), (20480, 64, 9), (20481, 64, 64), (20479, 1, 1),
                                         (1023, 7, 7), (1024, 64, 1), (1025, 2, 2), (4096, 33, 33), (4097, 64, 8), (8193, 5, 5)])
def test_dispatch_maps_in_one_launch(oracle, A, E, E_local):
    P.test_dispatch_index_only_short_lists(oracle, A, E, E_local)


# ----------------------------------------------------------------------------- one native call per layer
@pytest.mark.parametrize("T,k,E,E_local,dtype,fused,routing", [
    (1, 1, 8, 8, "bf16", True, "gate"), (16, 2, 64, 64, "bf16", True, "gate"), (300, 2, 33, 11, "bf16", True, "gate"),
    (1024, 1, 64, 64, "bf16", True, "ids"), (1025, 1, 64, 64, "bf16", True, "ids"), (512, 2, 64, 8, "bf16", True, "ids"),
    (77, 1, 8, 1, "bf16", True, "dropped"), (513, 1, 9, 9, "f32", True, "ids"), (200, 2, 5, 5, "f32", False, "gate"), (90, 2, 7, 7, "bf16", False, "ids")])
def test_layer_forward_is_its_calls(T, k, E, E_local, dtype, fused, routing):
    """moe_layer_forward writes what the separate calls write, maps included, also where it sorts without a dispatch launch."""
    _say(f"layer forward T={T} k={k} E={E} E_local={E_local} {dtype} fused={fused} {routing}")
    _layer_against_calls(T, k, E, E_local, dtype, fused, routing, 128, 192)


# a handful of rows: one to eight, up to sixteen tokens (gated by the first contraction) and past them, up to 64 assignments and past
# them; one to four tiles of experts; four and eight sums of the gate; blocks of 8 to 64 columns, one and several an expert
@pytest.mark.parametrize("T,k,E,E_local,d,f,routing", [
    (1, 1, 1, 1, 64, 64, "gate"), (1, 2, 2, 2, 1024, 4096, "gate"), (8, 1, 8, 8, 192, 64, "gate"), (4, 2, 17, 17, 2048, 320, "gate"), (9, 1, 16, 4, 2112, 128, "gate"),
    (16, 2, 33, 33, 64, 256, "gate"), (16, 1, 64, 64, 2048, 64, "gate"), (17, 1, 40, 40, 128, 448, "gate"), (5, 1, 32, 32, 4096, 64, "gate"),
    (3, 1, 8, 2, 1024, 2048, "ids"), (8, 1, 8, 8, 64, 8192, "ids"), (32, 2, 8, 8, 256, 512, "ids"), (64, 1, 3, 3, 128, 256, "ids"), (65, 1, 3, 3, 128, 256, "ids"),
    (7, 1, 64, 9, 128, 64, "dropped"), (2, 2, 64, 9, 128, 64, "dropped"), (16, 1, 1, 1, 512, 1024, "gate"),
    # the most gate weights that join the first contraction and the first that do not, either with the experts given
    (2, 1, 64, 64, 1600, 64, "gate"), (16, 2, 64, 64, 1664, 64, "gate"), (3, 1, 20, 20, 5440, 64, "gate"), (3, 1, 20, 20, 5504, 64, "gate"),
    (16, 1, 64, 8, 1664, 64, "ids"), (16, 2, 33, 33, 3008, 64, "ids"),
    # one row tile of a single expert and two, two experts past one tile
    (32, 1, 1, 1, 2048, 512, "gate"), (33, 1, 1, 1, 2048, 512, "gate"), (64, 1, 1, 1, 512, 2048, "gate"), (57, 1, 2, 2, 320, 2048, "gate")])
def test_layer_forward_of_a_few_rows(T, k, E, E_local, d, f, routing):
    _say(f"layer forward T={T} k={k} E={E} E_local={E_local} {d} x {f} {routing}")
    _layer_against_calls(T, k, E, E_local, "bf16", True, routing, d, f)


# the four calls in one: sorted by the first contraction (one to eight rows, up to 64, up to 1024; several row tiles a workgroup copies) and
# by a dispatch of its own, weighted by the second contraction (streamed, tiles of all kinds, fp32 in tiles of 16 and 64 rows) and by a combine
@pytest.mark.parametrize("T,k,E,E_local,dtype,routing,d,f", [
    (1, 1, 8, 8, "bf16", "gate", 64, 128), (8, 1, 8, 3, "bf16", "gate", 1024, 256), (16, 2, 33, 33, "bf16", "gate", 128, 64), (64, 1, 5, 5, "bf16", "ids", 192, 320),
    (7, 1, 64, 9, "bf16", "dropped", 128, 64), (65, 1, 20, 20, "bf16", "ids", 64, 192), (1024, 1, 64, 64, "bf16", "ids", 128, 64), (512, 2, 64, 48, "bf16", "gate", 64, 64),
    (1025, 1, 64, 64, "bf16", "ids", 64, 64), (300, 1, 3, 2, "bf16", "ids", 320, 576), (2000, 1, 7, 7, "bf16", "gate", 192, 128), (700, 1, 1, 1, "bf16", "gate", 1088, 256),
    (1100, 1, 9, 4, "bf16", "dropped", 64, 64), (40, 1, 6, 6, "f32", "ids", 36, 132), (1024, 1, 8, 4, "f32", "ids", 44, 812), (1025, 1, 4, 4, "f32", "ids", 64, 196),
    (512, 2, 5, 5, "f32", "gate", 64, 128)])
def test_unfused_layer_is_its_calls(T, k, E, E_local, dtype, routing, d, f):
    _say(f"unfused layer T={T} k={k} E={E} E_local={E_local} {dtype} {routing} {d} x {f}")
    _layer_against_calls(T, k, E, E_local, dtype, False, routing, d, f, ("x_sorted", "y_sorted"))


# the same where a first contraction in tiles sorts: one and eight assignments a thread, the longest list and the first with a dispatch launch; tiles of
# all kinds, whole and cut, reductions of one K tile, more columns of rows than of hidden activations (a tile copies several pieces of a row) and
# fewer than a piece; weights that are streamed (a dispatch launch); invalid ids, also all of them; the most tiles of a round and the first that are more; a share of the experts
@pytest.mark.parametrize("T,k,E,E_local,routing,d,f", [
    (60, 1, 1, 1, "gate", 4096, 4160), (257, 1, 1, 1, "ids", 64, 64), (512, 1, 2, 2, "gate", 128, 576), (513, 1, 9, 9, "ids", 1088, 64), (2047, 2, 64, 64, "gate", 64, 192),
    (2048, 2, 12, 12, "ids", 192, 1344), (4095, 1, 8, 8, "ids", 320, 1088), (4096, 1, 16, 16, "gate", 64, 4096), (4096, 1, 16, 16, "gate", 64, 4160), (4097, 1, 16, 16, "gate", 64, 320),
    (700, 1, 5, 5, "dropped", 64, 128), (1365, 2, 13, 13, "ids", 64, 64), (1500, 1, 33, 33, "gate", 448, 64), (1200, 2, 16, 16, "gate", 2048, 2112), (1500, 1, 64, 33, "ids", 448, 64)])
def test_layer_that_sorts_in_tiles_is_its_calls(T, k, E, E_local, routing, d, f):
    _say(f"layer in tiles T={T} k={k} E={E} E_local={E_local} {routing} {d} x {f}")
    _layer_against_calls(T, k, E, E_local, "bf16", False, routing, d, f, ("x_sorted", "y_sorted"))


# every expert resident and a map all the same: another order of them, and one that drops an expert's tokens and gives two others one expert; either activation
@pytest.mark.parametrize("T,k,E,dtype,routing,d,f,act,mapped", [
    (300, 1, 8, "bf16", "gate", 128, 576, 1, "permuted"), (700, 1, 9, "bf16", "ids", 64, 192, 0, "shared"), (2047, 2, 64, "bf16", "gate", 64, 192, 0, "permuted"),
    (2048, 2, 12, "bf16", "ids", 192, 1344, 1, "shared"), (4096, 1, 3, "bf16", "gate", 320, 1088, 1, "shared"), (257, 1, 1, "bf16", "ids", 64, 64, 1, "permuted"),
    (1024, 1, 8, "f32", "gate", 64, 256, 1, "permuted"), (1000, 1, 14, "f32", "ids", 44, 300, 0, "shared")])
def test_layer_that_sorts_by_a_map_of_resident_experts(T, k, E, dtype, routing, d, f, act, mapped):
    _say(f"layer with a {mapped} map T={T} k={k} E={E} {dtype} {routing} {d} x {f} act={act}")
    _layer_against_calls(T, k, E, E, dtype, False, routing, d, f, ("x_sorted", "y_sorted"), act=act, mapped=mapped)


# top-2 layers whose two rows of a token meet in the second contraction: up to eight rows, up to 64 and up to 1024; blocks of 8 to 64 columns and
# tiles of one and several row groups; tokens of which one or both assignments are dropped, and with the same expert twice ("ids"); the last
# shape of the separate calls that gets by with the reserved 16 MiB, the first that does not, and weights past the line
@pytest.mark.parametrize("T,E,E_local,dtype,fused,routing,d,f", [
    (1, 8, 8, "bf16", True, "gate", 64, 64), (4, 5, 5, "bf16", False, "ids", 1088, 128), (3, 64, 9, "bf16", True, "ids", 4096, 64), (5, 8, 3, "bf16", True, "gate", 192, 320),
    (32, 2, 2, "bf16", False, "gate", 704, 192), (31, 40, 13, "bf16", True, "ids", 128, 1088), (33, 3, 3, "bf16", True, "ids", 2112, 64), (128, 2, 1, "bf16", True, "ids", 64, 64),
    (100, 16, 16, "bf16", False, "ids", 512, 128), (512, 64, 64, "bf16", True, "gate", 128, 64), (511, 64, 40, "bf16", False, "ids", 64, 192), (60, 7, 2, "bf16", True, "dropped", 64, 64),
    (448, 64, 64, "bf16", False, "gate", 18688, 64), (448, 64, 64, "bf16", False, "gate", 18752, 64), (2, 2, 2, "bf16", True, "gate", 16448, 16384),
    (1, 2, 2, "f32", True, "gate", 4, 4), (27, 12, 12, "f32", True, "gate", 60, 156), (200, 9, 4, "f32", True, "ids", 44, 260), (512, 3, 3, "f32", True, "ids", 256, 1024),
    (512, 16, 16, "f32", True, "gate", 132, 1028), (90, 7, 7, "f32", False, "ids", 36, 64)])
def test_top2_rows_that_meet(T, E, E_local, dtype, fused, routing, d, f):
    _say(f"top-2 layer T={T} E={E} E_local={E_local} {dtype} fused={fused} {routing} {d} x {f}")
    _layer_against_calls(T, 2, E, E_local, dtype, fused, routing, d, f, () if fused else ("x_sorted", "y_sorted"))


@pytest.mark.parametrize("dtype,fused", [("bf16", True), ("bf16", False), ("f32", True)])
@pytest.mark.parametrize("T", [4, 20, 200])
def test_top2_rows_of_nans_meet(T, dtype, fused):
    """Also where every bit of the weights is set, as in a word that no row has reached yet, and with everything replayed from a graph.  (Separate
    calls in fp32 have a combine.)"""
    from paper_2401_08383_amd.pipeline import MoELayerRun

    g = torch.Generator(device="cuda")
    g.manual_seed(1650 + T)
    dt, bits = (torch.bfloat16, torch.int16) if dtype == "bf16" else (torch.float32, torch.int32)
    x, wg = (torch.randn(shape, device="cuda", generator=g).to(dt) for shape in ((T, 64), (4, 64)))
    w1, w2 = (torch.randn(shape, device="cuda", generator=g).to(dt) for shape in ((4, 128, 64), (4, 64, 128)))
    for w in (w1, w2):
        w[1].view(bits).fill_(-1)
    idx = torch.randint(0, 4, (T, 2), device="cuda", generator=g, dtype=torch.int32)
    idx[:4] = torch.tensor([[2, 3], [1, 2], [3, 1], [1, 1]])  # neither row, either one, both of NaNs
    run = MoELayerRun(x, wg, w1, w2, 2, True, topk_idx=idx, fused=fused)
    bad = (idx == 1).any(dim=1)
    # rows with eight bytes of set bits, as the separate calls leave them: fp32 has them, the conversion to bf16 makes 0xffc0 of these NaNs
    apart = MoELayerRun(x, wg, w1, w2, 2, True, topk_idx=idx)
    apart.step()
    torch.cuda.synchronize()
    assert bool((apart.y_sorted.view(torch.int64) == -1).any()) == (dtype == "f32")

    def look():
        torch.cuda.synchronize()
        assert bool(torch.isnan(run.out[bad]).all()) and bool(torch.isfinite(run.out[~bad]).all())
        return run.out[~bad].clone()

    run.step()
    first = look()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run.step()
    for _ in range(4):
        run.out.fill_(-7)
        graph.replay()
        assert torch.equal(look(), first)


def _layer_against_calls(T, k, E, E_local, dtype, fused, routing, d, f, more=(), act=0, mapped=None):
    from paper_2401_08383_amd.pipeline import MoELayerRun

    g = torch.Generator(device="cuda")
    g.manual_seed(1600 + T)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def rnd(*shape):
        return torch.randn(shape, device="cuda", generator=g).to(dt)

    expert_map = None
    if E_local < E:
        expert_map = torch.full((E,), -1, dtype=torch.int32, device="cuda")
        expert_map[torch.randperm(E, device="cuda", generator=g)[:E_local]] = torch.arange(E_local, dtype=torch.int32, device="cuda")
    elif mapped is not None:
        expert_map = torch.randperm(E, device="cuda", generator=g).int()
        if mapped == "shared":
            expert_map[0], expert_map[1] = -1, expert_map[2]
    idx = None
    if routing == "ids":
        idx = torch.randint(-1, E + 2, (T, k), device="cuda", generator=g, dtype=torch.int32)  # invalid ids among them
    elif routing == "dropped":
        idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    run = MoELayerRun(rnd(T, d), rnd(E, d), rnd(E_local, f, d), rnd(E_local, d, f), k, k > 1, expert_map=expert_map, topk_idx=idx, act=act, fused=fused)
    names = ["topk_idx", "topk_w", "src_of_sorted", "sorted_of_src", "expert_counts", "expert_offsets", "out", *more]

    def results(how):
        for n in names:
            getattr(run, n).fill_(-7)
        how()
        return [getattr(run, n).clone() for n in names]

    def calls():
        run.gate()
        run.dispatch()
        run.ffn()
        run.combine()

    ref = results(calls)
    got = results(run.step)
    for n, a, b in zip(names, got, ref):
        assert torch.equal(a, b), n
    run.x = rnd(T, d)  # an attribute that is assigned is used
    for n, a, b in zip(names, results(run.step), results(calls)):
        assert torch.equal(a, b), n


# one row a wavefront, several, 64 at a time and more than once round; the streamed contraction, tiles, fp32
@pytest.mark.parametrize("T,dtype", [(98, "bf16"), (1500, "bf16"), (7001, "bf16"), (250003, "bf16"), (700, "f32"), (40000, "f32")])
def test_rows_that_nobody_writes_are_cleared(T, dtype):
    _say(f"cleared rows T={T} {dtype}")
    g = torch.Generator(device="cuda")
    g.manual_seed(1700 + T)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn((T, 64), device="cuda", generator=g).to(dt)
    w1, w2 = (torch.randn(shape, device="cuda", generator=g).to(dt) for shape in ((2, 64, 64), (2, 64, 64)))
    idx = torch.randint(-1, 12, (T, 1), device="cuda", generator=g, dtype=torch.int32)
    maps = B.moe_dispatch(x, idx, 2, gather=False)
    out = torch.full_like(x, -7)
    B.moe_expert_ffn_fused(x, maps.src_of_sorted, maps.sorted_of_src, torch.ones((T, 1), device="cuda"), maps.expert_offsets, w1, w2, out=out)
    kept = maps.sorted_of_src.flatten()[:T] >= 0
    assert 0 < int(kept.sum()) < T // 4
    assert torch.equal(out[~kept], torch.zeros_like(out[~kept]))
    assert bool((out[kept] != -7).any(dim=1).all())


# ----------------------------------------------------------------------------- gate: ragged reductions, both tile heights
@pytest.mark.parametrize("T,d,E,k", [(1, 8, 1, 1), (17, 56, 16, 2), (16, 72, 17, 2), (33, 2056, 33, 1), (8191, 64, 64, 2), (8192, 200, 64, 2),
                                     (8200, 136, 17, 1), (40, 4096, 32, 2), (64 * 128 + 65, 1088, 48, 1)])
def test_gate_units_and_token_tiles(oracle, T, d, E, k):
    P.test_gate_topk_parity(oracle, "bf16", T, d, E, k, 1)


@pytest.mark.parametrize("T,d,E,k", [(16384, 8, 1, 1), (16385, 64, 64, 2), (16447, 200, 17, 2), (16448, 256, 33, 1), (16400, 320, 16, 2),
                                     (16384 + 63, 384, 48, 2), (16390, 2056, 9, 1), (20001, 136, 64, 1)])
def test_gate_of_a_long_batch(oracle, T, d, E, k):
    """From 64 * 256 tokens on: workgroups cut by the last token, reductions shorter than the ring, ragged ones, both sets of sums."""
    P.test_gate_topk_parity(oracle, "bf16", T, d, E, k, 1)


@pytest.mark.parametrize("d,E", [(64, 64), (1088, 40), (192, 8), (2112, 16), (2048, 17)])
def test_gate_of_a_long_batch_adds_as_the_shorter_one(d, E):
    """The same tokens in a shorter batch, through the other kernel: the same bits."""
    _say(f"gate long / shorter batch d={d} E={E}")
    g = torch.Generator(device="cuda")
    g.manual_seed(1900 + d)
    x = torch.randn((16384 + 31, d), device="cuda", generator=g).to(torch.bfloat16)
    w = torch.randn((E, d), device="cuda", generator=g).to(torch.bfloat16)
    first = 9000  # (between 8192 and 16384: four sums from 17 experts on, as in the long batch)
    for a, b in zip(B.moe_gate_topk(x, w, 2, True, True), B.moe_gate_topk(x[:first].contiguous(), w, 2, True, True)):
        assert torch.equal(a[:first], b)

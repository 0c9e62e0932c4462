"""GEMM tile shapes (128-, 64- and 32-row tiles, one or two wave sets sharing
the K loop) and tile orders: every shape on every case gives the oracle's
accumulators and outputs bit for bit, at K loops that end inside a stage, on
an odd granule, and with a group shorter than a stage."""
import numpy as np
import pytest
import torch

import oracle
import paper_2311_14114_amd as sq
import workloads

pytestmark = pytest.mark.gpu

CASES = [  # (M, N, K, a_frac, w_lo, w_hi, signed)
    (9, 130, 129, 0.5, 2, 4, True),        # two granules a group
    (33, 100, 64, 0.5, 1, 4, True),        # one granule a group
    (65, 300, 1000, 0.8, 2, 8, True),      # 13 + 4 granules: the last short K
    (64, 300, 1090, 0.8, 4, 8, False),     # 14 + 4: past it; zero points
    (130, 200, 2000, 0.97, 4, 4, True),    # 31 + 1
    (300, 1000, 777, 0.3, 3, 6, False),    # the wider group longer; weights the larger operand
    (1000, 140, 333, 0.8, 2, 4, True),     # activations the larger operand
    (100, 70, 1500, 0.8, 1, 8, True),      # no compiled pair: run-time containers
]


@pytest.mark.parametrize("shape", ["", "1", "3", "7", "8"])
@pytest.mark.parametrize("c", CASES, ids=lambda c: "x".join(map(str, c[:3])) + f"_w{c[4]}{c[5]}")
def test_tile_shapes(c, shape, monkeypatch):
    M, N, K, fa, wlo, whi, signed = c
    if shape:
        monkeypatch.setenv("SONIQ_GEMM_SHAPE", shape)
    case = workloads.generic(M, N, K, a_lo=4, a_hi=8, a_frac_lo=fa, w_lo=wlo, w_hi=whi, w_frac_lo=0.6,
                             a_signed=signed, a_abs=not signed, seed=M + N + K, name="tiles")
    print(f"[gpu] tiles {c} shape={shape or 'chosen'}", flush=True)
    w = sq.soniq_pack_weights(torch.from_numpy(case["W"]).cuda(), case["w_bits"], case["a_bits"], signed)
    act = sq.soniq_act_create(w, M)
    sq.soniq_quantize_act(act, torch.from_numpy(case["A"]).cuda())
    acc = torch.empty((w.S, M, N), dtype=torch.int32, device="cuda")
    guard = torch.full((M + 1, N + 3), 7.0, dtype=torch.bfloat16, device="cuda")
    Y = sq.soniq_mp_gemm(act, w, out=guard[:M, :N], acc=acc)
    torch.cuda.synchronize()
    r = oracle.run(case["A"], case["W"], case["a_bits"], case["w_bits"], signed)
    np.testing.assert_array_equal(acc.cpu().numpy(), r["acc"])
    np.testing.assert_array_equal(Y.contiguous().view(torch.int16).cpu().numpy().view(np.uint16), r["y_replay"])
    assert bool((guard[M] == 7.0).all()) and bool((guard[:, N:] == 7.0).all())


@pytest.mark.parametrize("B,C,H,W,N", [(1, 16, 7, 9, 40), (2, 48, 8, 8, 130), (3, 112, 14, 14, 96),
                                       (32, 64, 24, 24, 128), (33, 32, 24, 24, 128), (20, 16, 32, 32, 64),
                                       (2, 64, 20, 20, 70), (2, 96, 20, 20, 70)])
def test_conv_wave_sets(B, C, H, W, N):
    """The implicit convolution below and above one tile per CU and the K
    that two wave sets share, with taps of one to seven 16-channel units (a
    granule spans up to four taps)."""
    case = workloads.conv3x3(B, C, H, W, N, seed=B * C + H, name="conv_sets")
    print(f"[gpu] conv wave sets {B}x{C}x{H}x{W} -> {N}", flush=True)
    Wt = torch.from_numpy(case["W"]).reshape(N, C, 3, 3).contiguous().cuda()
    w = sq.soniq_pack_weights_conv3x3(Wt, case["w_bits"], case["a_bits"][::9].copy(), False, sign_nibbles=True)
    act = sq.soniq_act_create_conv3x3(w, B, H, W)
    sq.soniq_quantize_act_conv3x3(act, torch.from_numpy(case["X"]).cuda())
    M = B * H * W
    acc = torch.empty((w.S, M, N), dtype=torch.int32, device="cuda")
    Y = sq.soniq_mp_gemm(act, w, acc=acc)
    torch.cuda.synchronize()
    r = oracle.run(case["A"], case["W"], case["a_bits"], case["w_bits"], False)
    np.testing.assert_array_equal(acc.cpu().numpy(), r["acc"])
    np.testing.assert_array_equal(Y.view(torch.int16).cpu().numpy().view(np.uint16), r["y_replay"])


@pytest.mark.parametrize("with_acc", [True, False], ids=["acc", "y"])
@pytest.mark.parametrize("c", [  # (M, N, K, a_frac, w_lo, w_hi, group bits, input scale)
    (70, 200, 1000, 0.8, 2, 8, 512, 1.0),      # 13 + 4 granules: an odd narrow group
    (40, 130, 600, 0.2, 2, 4, 512, 1.0),       # 2 + 8
    (40, 130, 64, 1.0, 1, 4, 512, 1.0),        # one granule, sign weights
    # sign weights, whose stage is smaller than one load of the workgroup:
    # loads past it must stay in their own ring slot
    (37, 130, 450, 0.5, 1, 4, 512, 1.0),       # 4 + 4 granules: two stages a group
    (150, 300, 2300, 0.6, 1, 4, 512, 1.0),     # 22 + 15: more stages than slots, an odd wide granule
    (150, 300, 2240, 0.6, 1, 4, 1024, 1.0),    # 21 + 14: an odd narrow granule
    (70, 300, 2300, 0.6, 1, 1, 512, 1.0),      # no compiled pair: run-time containers
    (40, 130, 3000, 0.7, 4, 8, 1024, 1.0),     # blocks of four and two granules
    (40, 130, 700, 0.7, 2, 4, 512, 2.0 ** -104),  # scales too small for the folded shift
], ids=lambda c: "x".join(map(str, c[:3])) + f"_w{c[4]}{c[5]}_g{c[6]}")
def test_block_tiles(c, with_acc):
    """The tiles with sub-group scales: the 512-bit folds, the general hook,
    and both with accumulators asked for."""
    M, N, K, fa, wlo, whi, gbits, scale = c
    case = workloads.generic(M, N, K, a_lo=4, a_hi=8, a_frac_lo=fa, w_lo=wlo, w_hi=whi, w_frac_lo=0.6,
                             seed=M + N + K, name="block_tiles")
    A = case["A"] * np.float32(scale)
    print(f"[gpu] block tiles {c} acc={with_acc}", flush=True)
    w = sq.soniq_pack_weights(torch.from_numpy(case["W"]).cuda(), case["w_bits"], case["a_bits"], True,
                              act_group_bits=gbits)
    act = sq.soniq_act_create(w, M)
    sq.soniq_quantize_act(act, torch.from_numpy(A).cuda())
    acc = torch.empty((w.S, M, N), dtype=torch.int32, device="cuda") if with_acc else None
    Y = sq.soniq_mp_gemm(act, w, acc=acc)
    torch.cuda.synchronize()
    q_w, s_w = oracle.quantize_weights(case["W"], case["w_bits"])
    q_a, s_a, _, sub_of = oracle.quantize_act_grouped(A, case["a_bits"], True, gbits)
    racc = oracle.mac(q_a, q_w, sub_of, len(s_a))
    if with_acc:
        np.testing.assert_array_equal(acc.cpu().numpy(), racc)
    np.testing.assert_array_equal(Y.view(torch.int16).cpu().numpy().view(np.uint16),
                                  oracle.epilogue_replay(racc, s_a, s_w))

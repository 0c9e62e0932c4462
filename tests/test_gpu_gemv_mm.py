"""Decode batches on the fragment GEMV, with and without sub-group scales:
accumulators and outputs bit-exact against the oracle, at the edges of its
rounds (chunks per wave), of its rows (1 to 8), of odd granule counts and of
every weight container, and rows longer than one launch's staging."""
import numpy as np
import pytest
import torch

import oracle
import paper_2311_14114_amd as sq
import workloads

pytestmark = pytest.mark.gpu

CASES = [  # (M, N, K, a_lo, a_hi, a_frac, w_lo, w_hi, signed, group bits)
    (2, 40, 64, 4, 4, 1.0, 2, 4, True, 0),            # one granule, one group
    (5, 40, 129, 4, 8, 0.5, 1, 4, True, 0),           # sign weights above 4 rows
    (8, 40, 700, 3, 6, 0.8, 1, 1, False, 0),
    (3, 40, 3584, 4, 8, 1.0, 4, 8, True, 0),          # 56 narrow granules: one full round
    (3, 40, 3650, 4, 8, 0.98, 8, 8, False, 0),        # and past it; zero points
    (4, 40, 3712, 4, 4, 1.0, 2, 4, True, 0),          # 58: the second wave's only extra granule
    (2, 40, 3840, 4, 4, 1.0, 2, 8, True, 0),          # 60: each wave has one
    (7, 40, 1100, 4, 8, 0.02, 3, 6, True, 0),         # 17 wide granules: past a round's 16
    (4, 40, 1536, 4, 4, 1.0, 2, 4, True, 0),          # 24 narrow granules: a full short round
    (8, 40, 1600, 4, 4, 1.0, 4, 8, True, 0),          # and 25
    (3, 40, 560, 4, 8, 0.05, 1, 8, True, 0),          # 9 wide granules; 8 below
    (6, 40, 530, 4, 8, 0.05, 2, 8, False, 0),
    (5, 40, 1530, 4, 4, 1.0, 2, 8, True, 512),
    (2, 40, 1660, 4, 4, 1.0, 4, 4, True, 512),
    (7, 40, 530, 4, 8, 0.05, 3, 6, True, 512),
    (8, 33, 11008, 4, 8, 0.8, 2, 4, True, 0),         # three rounds
    (1, 33, 60000, 4, 8, 0.8, 4, 8, True, 0),         # a row too long to stage
    (1, 40, 700, 4, 8, 0.8, 1, 4, True, 512),
    (2, 40, 64, 4, 4, 1.0, 2, 4, True, 512),
    (4, 40, 2000, 4, 8, 0.8, 2, 8, True, 512),
    (8, 40, 3711, 4, 8, 0.97, 4, 8, True, 512),       # an odd narrow granule count
    (8, 33, 11008, 4, 8, 0.8, 2, 4, True, 512),       # the most products that fit
    (3, 40, 2066, 4, 8, 0.2, 1, 8, True, 0),          # wide rounds: 26 wide granules in one
    (2, 40, 6650, 3, 6, 0.2, 2, 8, False, 0),         # and in three
    (8, 40, 3000, 4, 8, 0.05, 4, 8, True, 0),         # 45 wide granules: the widest round
    (5, 40, 3300, 4, 8, 0.02, 2, 4, True, 512),       # past it: 51
    (4, 8300, 2420, 4, 8, 0.8, 2, 4, True, 0),        # several rounds of one chunk
    (1, 40, 1757, 3, 6, 0.95, 3, 6, True, 1024),
    (2, 40, 2000, 4, 8, 0.2, 1, 4, True, 1536),       # three chunks per block, partial last blocks
    (8, 40, 1000, 4, 8, 0.5, 2, 8, True, 65536),      # one block a group
    (6, 40, 2500, 4, 8, 0.7, 2, 4, True, 1024),       # two chunks per block
    (3, 40, 5000, 3, 7, 0.7, 4, 4, False, 2048),      # four, unsigned
]


@pytest.mark.parametrize("with_acc", [True, False], ids=["acc", "y"])
@pytest.mark.parametrize("c", CASES, ids=lambda c: "x".join(map(str, c[:3])) + f"_w{c[6]}{c[7]}_g{c[9]}")
def test_gemv_mm(c, with_acc):
    M, N, K, alo, ahi, fa, wlo, whi, signed, gbits = c
    case = workloads.generic(M, N, K, a_lo=alo, a_hi=ahi, a_frac_lo=fa, w_lo=wlo, w_hi=whi, w_frac_lo=0.6,
                             a_signed=signed, a_abs=not signed, seed=3 * M + K, name="gemv_mm")
    print(f"[gpu] gemv_mm {c} acc={with_acc}", flush=True)
    w = sq.soniq_pack_weights(torch.from_numpy(case["W"]).cuda(), case["w_bits"], case["a_bits"], signed,
                              act_group_bits=gbits)
    act = sq.soniq_act_create(w, M)
    sq.soniq_quantize_act(act, torch.from_numpy(case["A"]).cuda())
    acc = torch.empty((w.S, M, N), dtype=torch.int32, device="cuda") if with_acc else None
    Y = sq.soniq_mp_gemm(act, w, acc=acc)
    torch.cuda.synchronize()
    q_w, s_w = oracle.quantize_weights(case["W"], case["w_bits"])
    if gbits:
        q_a, s_a, _, sub_of = oracle.quantize_act_grouped(case["A"], case["a_bits"], signed, gbits)
        racc = oracle.mac(q_a, q_w, sub_of, len(s_a))
    else:
        r = oracle.run(case["A"], case["W"], case["a_bits"], case["w_bits"], signed)
        s_a, racc = r["s_a"], r["acc"]
    if with_acc:
        np.testing.assert_array_equal(acc.cpu().numpy(), racc)
    np.testing.assert_array_equal(Y.view(torch.int16).cpu().numpy().view(np.uint16),
                                  oracle.epilogue_replay(racc, s_a, s_w))

"""Activation quantizers on rows of any length, stride and alignment: codes,
scales, accumulators and outputs against the oracle (bit-exact), at the
edges of the four-value pieces a row is cut into, of the small-batch launch
(rows, values per thread) and of the single pass and its two-pass form."""
import numpy as np
import pytest
import torch

import oracle
import paper_2311_14114_amd as sq
import workloads

pytestmark = pytest.mark.gpu

CASES = [  # (M, N, K, a_lo, a_hi, signed, lda pad, first element, group bits)
    (1, 40, 3, 4, 8, True, 0, 0, 0),          # shorter than a piece
    (1, 40, 4, 4, 8, True, 1, 1, 0),          # one piece
    (3, 40, 5, 4, 8, True, 0, 3, 0),          # two pieces overlapping in three values
    (8, 64, 255, 4, 8, True, 0, 1, 0),
    (8, 64, 2049, 4, 8, False, 2, 0, 0),      # one piece past 512 threads
    (5, 64, 4097, 4, 8, True, 1, 2, 0),       # four pieces a thread
    (1, 33, 16383, 4, 8, True, 0, 1, 0),      # the longest row of the small batch
    (1, 33, 16385, 4, 8, True, 0, 1, 0),      # and past it
    (64, 64, 1023, 3, 6, False, 1, 1, 0),     # the most rows of the small batch
    (65, 64, 1023, 3, 6, False, 1, 1, 0),     # and past it: two passes
    (9, 64, 7291, 4, 8, True, 0, 2, 0),
    (7, 48, 510, 1, 8, True, 1, 0, 0),        # a sign group
    (70, 48, 509, 1, 4, True, 0, 1, 0),
    (301, 96, 4091, 3, 6, False, 0, 0, 0),    # two passes, two rows a workgroup in the first
    (1100, 64, 1001, 4, 8, True, 3, 1, 0),    # four rows
    (1030, 32, 770, 4, 8, False, 1, 0, 0),
    (2050, 32, 513, 4, 8, True, 1, 1, 0),     # eight rows
    (7169, 32, 149, 4, 8, False, 0, 3, 0),    # many short rows: the single pass
    (2, 40, 1500, 4, 8, True, 0, 0, 0),       # small batches: two, four, one row in flight
    (4, 40, 1902, 4, 8, False, 1, 1, 0),
    (1, 40, 3001, 4, 8, True, 0, 0, 0),
    (2, 40, 3001, 3, 6, True, 0, 2, 0),
    (1, 40, 5000, 4, 8, True, 0, 0, 0),
    (1, 48, 130, 4, 8, True, 0, 0, 512),      # block maxima of few short rows: the longest, and past it
    (8, 48, 1024, 4, 8, True, 0, 0, 512),
    (7, 48, 1023, 3, 6, False, 1, 1, 1024),
    (8, 48, 1025, 4, 8, True, 0, 0, 512),
    (9, 48, 500, 4, 8, True, 0, 0, 512),
    (1, 48, 1027, 4, 8, True, 0, 1, 512),
    (8, 48, 4099, 4, 8, True, 1, 1, 512),
    (33, 48, 1981, 4, 8, True, 0, 3, 512),
    (64, 48, 300, 2, 8, True, 0, 0, 1024),
    (300, 48, 4095, 4, 8, True, 0, 1, 512),   # single pass with blocks
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: "x".join(map(str, c[:3])) + f"_g{c[8]}_o{c[7]}")
def test_rows(c):
    M, N, K, lo, hi, signed, pad, first, gbits = c
    case = workloads.generic(M, N, K, a_lo=lo, a_hi=hi, a_frac_lo=0.7, w_lo=2, w_hi=4, w_frac_lo=0.6,
                             a_signed=signed, a_abs=not signed, seed=M + 7 * K, name="rows")
    print(f"[gpu] rows {c}", flush=True)
    buf = torch.full((first + M * (K + pad),), 1e30, dtype=torch.float32, device="cuda")
    A = buf.as_strided((M, K), (K + pad, 1), first)
    A.copy_(torch.from_numpy(case["A"]))
    w = sq.soniq_pack_weights(torch.from_numpy(case["W"]).cuda(), case["w_bits"], case["a_bits"], signed,
                              act_group_bits=gbits)
    act = sq.soniq_act_create(w, M)
    acc = torch.empty((w.S, M, N), dtype=torch.int32, device="cuda")
    Y = sq.soniq_quantize_mp_gemm(act, w, A, acc=acc)
    torch.cuda.synchronize()
    q_a, s_a = sq.soniq_act_unpack_debug(act)
    q_w, s_w = oracle.quantize_weights(case["W"], case["w_bits"])
    if gbits:
        rq, rs, _, sub_of = oracle.quantize_act_grouped(case["A"], case["a_bits"], signed, gbits)
        racc = oracle.mac(rq, q_w, sub_of, len(rs))
    else:
        r = oracle.run(case["A"], case["W"], case["a_bits"], case["w_bits"], signed)
        rq, rs, racc = r["q_a"], r["s_a"], r["acc"]
    np.testing.assert_array_equal(s_a, rs)
    np.testing.assert_array_equal(q_a, rq)
    np.testing.assert_array_equal(acc.cpu().numpy(), racc)
    np.testing.assert_array_equal(Y.view(torch.int16).cpu().numpy().view(np.uint16),
                                  oracle.epilogue_replay(racc, rs, s_w))


@pytest.mark.parametrize("M", [63, 129, 513, 2047, 2049, 4097, 7169, 8193])
def test_two_pass_rows_per_workgroup(M, monkeypatch):
    """Each row count of the first pass's workgroups (2, 4, 8, 16), with
    batches that end inside a workgroup and inside a 16-row block."""
    case = workloads.generic(M, 32, 1100, a_lo=3, a_hi=8, a_frac_lo=0.6, w_lo=2, w_hi=4, w_frac_lo=0.5,
                             a_signed=False, a_abs=True, seed=M, name="two_pass")
    monkeypatch.setenv("SONIQ_ACT_COOP", "0")
    print(f"[gpu] two pass M={M}", flush=True)
    case["A"][M - 1, 7] = 9.0  # the last row holds both maxima
    case["A"][M - 1, 8] = 9.5
    w = sq.soniq_pack_weights(torch.from_numpy(case["W"]).cuda(), case["w_bits"], case["a_bits"], False)
    act = sq.soniq_act_create(w, M)
    sq.soniq_quantize_act(act, torch.from_numpy(case["A"]).cuda())
    torch.cuda.synchronize()
    q_a, s_a = sq.soniq_act_unpack_debug(act)
    r = oracle.run(case["A"][:], case["W"][:1], case["a_bits"], case["w_bits"][:1], False)
    np.testing.assert_array_equal(s_a, r["s_a"])
    np.testing.assert_array_equal(q_a, r["q_a"])

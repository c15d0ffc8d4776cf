"""Host-side checks of the measurement code (no GPU): the bench counts every
scored round once, in the scoring kernel's entry or as the next-round scoring
of the kernel that culls and refines; the counter summary's rates."""
import csv

import pytest

import bench
from paper_1801_08361_amd import rocprof_summary as rs


@pytest.mark.parametrize("n_hyp,n_valid,batch_pixels,scored", [
    (1024, 1000, 500, 6),       # rounds 6-9 are scored by the round before
    (256, 256, 64, 3),
    (64, 40, 2000, 4),          # 8 positions are the first with few enough workgroups
    (2, 2, 64, 1)])             # one round: no next one
def test_scoring_is_counted_once(n_hyp, n_valid, batch_pixels, scored):
    rounds = max(1, (n_hyp - 1).bit_length())
    n_rounds = max(1, (n_valid - 1).bit_length())
    res = [dict(mode_evals=12345, pair_evals=678, n_valid=n_valid, n_rounds=n_rounds)]
    kernels = {"k_b_score": (2.0, min(scored, rounds)), "k_b_cull_refine": (3.0, 6)}
    r = bench.rooflines(kernels, res, [(100, 5, False, n_hyp)], batch_pixels=batch_pixels)
    total = 12345 * bench.FLOP_PER_MODE_TERM + 678 * bench.FLOP_PER_PAIR
    lives = [n_valid]
    while len(lives) < n_rounds:
        lives.append((lives[-1] + 1) // 2)
    by_score = r["k_b_score"]["work_per_launch"] * min(scored, rounds)
    assert by_score == pytest.approx(total * sum(lives[:scored]) / sum(lives))
    nxt = r["k_b_cull_refine"].get("next_scoring")
    if sum(lives[scored:]) == 0:
        assert nxt is None
        return
    assert by_score + nxt["flops_per_launch"] * 6 == pytest.approx(total)
    assert nxt["tflops"] == pytest.approx(nxt["flops_per_launch"] * 6 / 3.0e-3 / 1e12)
    share = sum(lives[scored:]) / sum(lives)
    ids = sum(lives[scored:]) * (batch_pixels * (16 + 8 * 5 + 4) + 4 * ((batch_pixels + 7) // 8))
    assert nxt["bytes_per_launch"] * 6 == pytest.approx(12345 * share * 48 + ids)


def test_rates(tmp_path):
    def put(d, name, header, rows):
        (tmp_path / d).mkdir()
        with open(tmp_path / d / name, "w", newline="") as f:
            csv.writer(f).writerows([header] + rows)
    hdr = ["Kernel_Name", "Counter_Name", "Counter_Value"]
    k = "void rl::(anonymous namespace)::k_x<8>(rl::A)"
    put("sq", "s_counter_collection.csv", hdr, [[k, "SQ_INSTS_VALU", 1024 * 600], [k, "SQ_INSTS_VMEM_RD", 256 * 120],
                                                [k, "SQ_INSTS_LDS", 3000], [k, "SQ_LDS_BANK_CONFLICT", 1500],
                                                [k, "SQ_WAVES", 1000], ["at::other", "SQ_WAVES", 7]])
    put("tcp", "t_counter_collection.csv", hdr, [[k, "TCP_TOTAL_CACHE_ACCESSES_sum", 256 * 4800],
                                                 [k, "TCP_TCC_READ_REQ_sum", 256 * 1200]])
    put("st", "p_kernel_stats.csv", ["Name", "Calls", "TotalDurationNs", "AverageNs", "MinNs", "MaxNs"],
        [[k, 2, 2000, 1000, 1, 1], ["at::other", 1, 1, 1, 1, 1]])
    text = rs.rates(str(tmp_path / "sq"), str(tmp_path / "tcp"), str(tmp_path / "st"))
    # 2400 cycles: 4 x 600 of them busy a SIMD, 20 per load, 2 L1 accesses a cycle
    assert text.splitlines()[2:] == ["| k_x<8> | 1.00 | 1,000 | 100.0 % | 20.0 | 2.000 | 0.250 | 3 | 0.50 |"]

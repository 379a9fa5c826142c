"""The counter summary's choice of kernels (no device): its default takes the
FP32 one-site H_eff GEMM alone from a file that holds several precisions."""
import csv
import json

from paper_2005_06104_amd import tracesum

NS = "void (anonymous namespace)::"
FP32 = NS + "gemm_split_kernel<(anonymous namespace)::SplitTile<3, 64, 64, 2, 2, 2, true, false>, false, false, 1>(int, int)"
BF16 = NS + "gemm_split_kernel<(anonymous namespace)::SplitTile<1, 64, 64, 2, 2, 3, true, false>, false, false, 1>(int, int)"
FP64 = NS + "gemm_direct_kernel<(anonymous namespace)::DirectTile<2, 2, 2, 2, 1, 4, true, false>, false, false, 1>(int, int)"
ENV = NS + "gemm_split_kernel<(anonymous namespace)::SplitTile<3, 64, 64, 2, 2, 2, true, false>, false, false, 0>(int, int)"


def test_default_kernel_is_one_family(tmp_path, capsys):
    p = tmp_path / "counters.csv"
    with open(p, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Correlation_Id", "Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
        for i, (k, v) in enumerate([(FP32, 10.0), (BF16, 1000.0), (FP64, 7000.0), (ENV, 300.0), (FP32, 30.0)]):
            w.writerow([i, i, k, "FETCH_SIZE", v])
    tracesum.main([str(p), "--counters", "--marker", "none"])
    out = json.loads(capsys.readouterr().out)
    assert out["dispatches"] == 2 and out["avg"]["FETCH_SIZE"] == 20.0 and out["kernels"] == [FP32]
    tracesum.main([str(p), "--counters", "--marker", "none", "--kernel", "gemm_", "--kernel", ", 1>("])
    assert json.loads(capsys.readouterr().out)["kernels"] == sorted([FP32, BF16, FP64])

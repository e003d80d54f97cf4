"""profsum.call_bytes on made-up counter databases: every kernel that a
library call launches is found once, by its name in a profiler run."""
import sqlite3

import profsum

# kernels of one linear-attention forward and gradient call (32768 steps, 4
# heads), as the profiler names them, with bytes per dispatch in KiB
KERNELS = {
    "memoroid::linattn_summary_kernel(memoroid::LinSummaryArgs)": 1,
    "void memoroid::state_scan_kernel<4, false>(memoroid::LinScanArgs)": 2,
    "void memoroid::linattn_output_kernel<false>(memoroid::LinOutputArgs)": 4,
    "void memoroid::linattn_dq_kernel<false>(memoroid::LinBwdArgs)": 8,
    "void memoroid::state_scan_kernel<4, true>(memoroid::LinScanArgs)": 16,
    "void memoroid::linattn_dkv_kernel<false>(memoroid::LinBwdArgs)": 32,
}


def _db(path, kernels):
    con = sqlite3.connect(path)
    con.execute("create table pmc_events (name text, counter_value real)")
    # the calibration copy reads its true size: a scale of one
    con.execute("insert into pmc_events values (?, ?)", (profsum.COPY_KERNEL, profsum.COPY_BYTES / 1024.0))
    for name, kib in kernels.items():
        for _ in range(3):
            con.execute("insert into pmc_events values (?, ?)", (name, kib))
    con.commit()
    con.close()
    return str(path)


def test_linear_attention_calls_find_each_kernel_once(tmp_path):
    fetch, write = _db(tmp_path / "f.db", KERNELS), _db(tmp_path / "w.db", KERNELS)
    got = profsum.call_bytes(9, fetch, write)
    assert got == {"linattn_fwd": 2 * 7 * 1024, "linattn_bwd": 2 * 59 * 1024}
    fwd = {k: v for k, v in KERNELS.items() if v in (1, 2, 4)}
    assert profsum.call_bytes(3, _db(tmp_path / "f3.db", fwd), _db(tmp_path / "w3.db", fwd)) == {
        "linattn_fwd": 2 * 7 * 1024}

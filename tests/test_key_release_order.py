"""The split CG update's hand-over, in the code built for gfx950 (CPU only).

key_cg_split_kernel stores Ap with several waves of a block, and one thread then
releases the block's part for the block that finishes last, on whatever die that
runs.  A workgroup barrier does not wait for global stores, so each storing wave
has to drain its own before the barrier that the releasing thread passes: in every
instance an s_waitcnt vmcnt(0) stands between the store of Ap (the last 16-byte
store before the L2 write-back) and the next s_barrier."""
import os
import re
import subprocess

import pytest

from paper_2605_31105_amd import build as B


def test_ap_stores_drain_before_the_release(tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("hipcc missing")
    out = tmp_path / "key.s"
    subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-device-only", "-S",
                    os.path.join(B.CSRC, "key.hip"), "-o", str(out)],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    kernels = re.findall(r"^(_Z\S*key_cg_split_kernel\S*):(.*?)^\.Lfunc_end", out.read_text(),
                         re.S | re.M)
    assert len(kernels) == 6   # 32, 64 and 128 rows, head dimension 64 and 128
    for name, body in kernels:
        code = [line.split(";")[0].strip() for line in body.splitlines()]
        release = next(i for i, c in enumerate(code) if c.startswith("buffer_wbl2"))
        store = max(i for i in range(release) if code[i].startswith("global_store_dwordx4"))
        barrier = next(i for i in range(store, release) if code[i].startswith("s_barrier"))
        drains = [c for c in code[store:barrier] if re.match(r"s_waitcnt .*vmcnt\(0\)", c)]
        assert drains, "%s: stores of Ap not drained before the barrier" % name

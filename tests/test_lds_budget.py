"""LDS of the decode kernels that are launched next to resident prefill workgroups."""
import os
import re
import subprocess


def lds_of(source):
    """{kernel: (bytes of LDS, vector registers)} as the compiler reports them with the library's flags."""
    from paper_2512_03416_amd import build as B
    r = subprocess.run([B.HIPCC] + B.FLAGS + ["-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c", os.path.join(B.CSRC, source), "-o", os.devnull],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found, name, regs = {}, None, 0
    for line in r.stderr.splitlines():
        for what, value in re.findall(r"(Function Name| VGPRs|LDS Size \[bytes/block\]): (\S+)", line):
            if what == "Function Name":
                name = value
            elif what == " VGPRs":
                regs = int(value)
            else:
                found[name] = (int(value), regs)
    return found


def test_decode_workgroups_fit_next_to_a_resident_prefill_workgroup():
    """A CU has 160 KB: a decode workgroup of head dim 128 that fits by its registers (128 a lane next to two waves of 192) has to
    fit into what the resident workgroup leaves, or the scan waits for the tiles.  (decode_kernel: the option
    decode_prefetch_tiles; the alone and fused forms never run there.)"""
    resident = [v for k, v in lds_of("ts_kernels_mixed.hip").items() if "prefill_resident_kernel" in k]
    assert len(resident) == 3
    left = 160 * 1024 - max(lds for lds, _ in resident)
    kernels = {k: v for k, v in lds_of("ts_kernels_decode.hip").items()
               if "Li128E" in k and re.search(r"decode_kernel(_lean|_lean_merging)?I", k) and v[1] <= 128}
    assert len(kernels) == 5                               # lean and lean_merging of both caches, three tiles of an e4m3 cache
    for name, (lds, _) in kernels.items():
        assert lds <= left, (name, lds, left)

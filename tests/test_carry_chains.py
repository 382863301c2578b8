"""The carry chains of the 128-bit sums and of the lazy quotients: on the host
with operands that carry everywhere, and, for the instructions that the device
runs, the distance between each mask's writer and its reader."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native")
# the wait states that the compiler keeps on gfx950 between a vector instruction that
# writes a mask (carry, select) and one that reads it
MASK_WAIT = 2


def test_mac_carry_chain_host_exact(tmp_path):
    exe = str(tmp_path / "mac")
    subprocess.check_call(["hipcc", "-O2", "-std=c++17", os.path.join(NATIVE, "mac_carry_test.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert " 0 failures" in out.stdout


def mask_reads(text):
    """(wait states since the mask was written, the reading instruction) of every
    vector instruction of an assembly listing that reads a mask written by a
    vector instruction of the same block."""
    at, written, found = 0, {}, []
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if line.endswith(":"):
            written = {}
        m = re.match(r"([sv]_\w+|global_\w+|flat_\w+|ds_\w+|buffer_\w+|scratch_\w+)\s*(.*)", line)
        if not m:
            continue
        op, args = m.group(1), [a.strip() for a in re.split(r",(?![^\[]*\])", m.group(2))]
        read = wrote = None
        if re.match(r"v_(addc|subb|subbrev)_co", op):
            wrote, read = args[1], args[4]
        elif op.startswith("v_cndmask"):
            read = args[3] if len(args) > 3 else "vcc"
        elif re.match(r"v_(add|sub|subrev)_co|v_mad_[ui]64", op):
            wrote = args[1]
        elif op.startswith("v_cmp"):
            wrote = args[0]
        elif op.startswith("s_") and args[0] in written:
            del written[args[0]]  # the scalar unit's result, which the hardware waits for
        if read in written:
            found.append((at - written[read] - 1, line))
        if wrote and (wrote == "vcc" or wrote.startswith("s[")):
            written[wrote] = at
        at += int(args[0], 0) + 1 if op == "s_nop" else 1
    return found


def test_mask_readers_wait_for_their_writers(tmp_path):
    lst = str(tmp_path / "chains.s")
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                           "-packed-fp32-ops", "--offload-device-only", "-S", os.path.join(NATIVE, "carry_chains.hip"),
                           "-o", lst], stderr=subprocess.DEVNULL)
    reads = mask_reads(open(lst).read())
    assert sum("v_addc_co" in r for _, r in reads) >= 3   # the sum's chain
    assert sum("v_cndmask" in r for _, r in reads) >= 2   # the quotients' carries (barrett_sum, shoup_add)
    assert not [r for r in reads if r[0] < MASK_WAIT]

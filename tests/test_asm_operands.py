"""The event loops written out in assembly, compiled apart from their kernels (no GPU needed): a register that the
asm writes before it has read all its inputs is never an input's.  The probe gives the compiler every occasion: the low
registers are taken, the inputs die at the asm, and those written in it start as copies of those that are only read."""
import os
import re
import subprocess

import pytest

from paper_1409_6948_amd import build as B

PROBE = r"""
#include <hip/hip_runtime.h>
#include <stdint.h>
constexpr int kDigestBatch = 64;
%s
__global__ void __launch_bounds__(64) probe(const double* __restrict__ in, const int* __restrict__ num, double* out,
                                            int s_gridb, int s_inv_g32, int s_top, int limit, int key_in, double mid,
                                            double inner, double s_sig2, double s_inv_b, double s_reach, double s_L,
                                            double s_inv_L) {
  const int lane = threadIdx.x;
  double2 p = make_double2(in[lane], in[lane + 64]);
  double ax = in[lane + 128], ay = in[lane + 192], nrem = s_reach, dacc = mid, sum = in[lane + 256];
  double dx = in[lane + 320], dy = in[lane + 384], guard = in[lane + 448], s;
  int rec_lo = num[lane], rec_hi = num[lane + 64], rec_tag = num[lane + 128], m = num[lane + 192];
  const int pos_at = num[lane + 256], meta_at = num[lane + 320], own_loc_at = num[lane + 384], loff = num[lane + 448];
  const int slot_of_at = own_loc_at, lx = loff, ly = num[lane + 512], s_nb = s_gridb, s_inv_n32 = s_inv_g32;
  const double s_mid = mid, s_inner = inner;
  int widx = loff, wsl = loff, woff = loff, upos_at = pos_at, uslot_at = meta_at;
  int a_slot = s_gridb, a_lidx = s_top, n_ring = limit, offx = s_top, offy = s_inv_g32, n_frozen = s_gridb, a = s_top;
  int key, key_min, full, a_t, a_u, a_next, a_slo, a_shi, a_expect;
  double acc = sum;
  uint64_t a_mask;
  %s;
  const double v[] = {p.x, p.y, ax, ay, nrem, dacc, sum, acc, dx, dy, guard, s, (double)(rec_lo + rec_hi + rec_tag + m),
                      (double)(widx + wsl + woff + upos_at + uslot_at), (double)(a_slot + a_lidx + n_ring + a),
                      (double)(offx + offy + n_frozen), (double)(key + key_min + full)};
  double t = 0.0;
  for (double q : v) t += q;
  out[lane] = t;
}
"""

OUT = ["kmin", "full", "a_slot", "a_lidx", "mask", "t", "u", "next", "slo", "shi", "expect"]
WALLED = ["pos", "meta", "own_loc", "loff", "mid", "inner", "sig2", "inv_b", "reach", "gridb", "inv_g32", "top", "limit",
          "low31"]
# the loop, its operands that are written, those that are only read
LOOPS = {
    "walled": ('EC_LOOP("", "", "6f", EC_REFLECTION, )', OUT + ["woff", "offx", "offy", "n_frozen"], WALLED),
    "rejection": ('EC_LOOP(EC_UNDO_LOG, EC_UNDO_STEP, "2f", "", EC_UNDO_OPERANDS)',
                  OUT + ["woff", "offx", "offy", "n_frozen", "uslot", "upos"], WALLED),
    "periodic": ("EC_LOOP_PERIODIC", OUT, ["pos", "meta", "own_loc", "lx", "ly", "mid", "inner", "sig2", "inv_b", "L",
                                           "inv_L", "gridb", "inv_g32", "offx", "offy"]),
}


def _loops_of_the_source():
    text = open(os.path.join(B.CSRC, "ec_kernels.hip")).read()
    a, b = text.index("#define EC_W(x)"), text.index("// Both components of (x, y) / den")
    return text[a:b]


def _registers(word):
    """'v[64:65]' or 'v64' -> {('v', 64), ...}; a literal -> empty set"""
    r = re.fullmatch(r"([vs])\[(\d+):(\d+)\]", word)
    if r:
        return {(r[1], k) for k in range(int(r[2]), int(r[3]) + 1)}
    r = re.fullmatch(r"([vs])(\d+)", word)
    return {(r[1], int(r[2]))} if r else set()


@pytest.mark.parametrize("loop", list(LOOPS))
def test_inputs_of_the_written_out_loop_are_in_no_register_that_it_writes(loop, tmp_path):
    call, written, read = LOOPS[loop]
    names = written + read
    macros = _loops_of_the_source()
    # a comment line of the asm lists the operands' registers
    line = 'EC_W("; operands ' + " ".join(f"{n}=%[{n}]" for n in names) + '") EC_FOUR('
    start = macros.index("#define EC_LOOP_PERIODIC" if loop == "periodic" else "#define EC_LOOP(")
    at = macros.index("EC_FOUR(", start)
    macros = macros[:at] + line + macros[at + len("EC_FOUR("):]
    # its own fixed registers, those of the outputs among them
    end = macros.index("\n\n", at) if "\n\n" in macros[at:] else len(macros)
    end = min([k for k in (macros.find("// The rejection variant's", at), end) if k > 0])
    block = macros[at:end]
    fixed = set()
    for word in re.findall(r"\{(v\[\d+:\d+\]|v\d+|s\[\d+:\d+\])\}", block):
        fixed |= _registers(word)
    clobbers = block[block.index('"vcc", "scc"'):]
    for word in re.findall(r'"([vs]\d+)"', clobbers):
        fixed |= _registers(word)
    # the registers below v96 that are still free are taken
    taken = ", ".join(f'"v{k}"' for k in range(96) if ("v", k) not in fixed)
    macros = macros[:at] + block.replace('"vcc", "scc"', taken + ', "vcc", "scc"', 1) + macros[end:]
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE % (macros, call))
    r = subprocess.run([B.HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "-S",
                        "-o", str(out), str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found = re.findall(r"; operands (.*)", out.read_text())
    assert len(found) == 1
    where = dict(w.split("=") for w in found[0].split())
    assert set(where) == set(names)
    seen = {}
    for name, word in where.items():
        regs = _registers(word)
        assert regs or name == "low31", (name, word)  # (low31 may be a literal)
        assert not regs & fixed, f"[{name}] is {word}, which the asm writes or keeps for another operand"
        for g in regs:
            assert g not in seen or (name in read and seen[g] in read), f"[{name}] and [{seen[g]}] share {word}"
            seen[g] = name

"""Scalar and packed instructions of every source's gfx950 assembly.

Scalar instructions are checked against a list of those that may appear: the
arithmetic, control and wait instructions, and of the ones that touch memory
the plain loads.  So memory is written by vector instructions only.  Packed
float32 arithmetic (which the build turns off) may not appear at all."""

import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2111_11215_amd import build as B

LOADS = {f"s_load_dword{n}" for n in ("", "x2", "x3", "x4", "x8", "x16")} | \
    {f"s_buffer_load_dword{n}" for n in ("", "x2", "x3", "x4", "x8", "x16")}
ARITHMETIC = re.compile(
    r"s_(abs|add|addc|addk|and|andn1|andn2|ashr|bcnt0|bcnt1|bfe|bfm|bitcmp0|bitcmp1|bitset0|bitset1|brev|cmov|cmovk|"
    r"cmp|cmpk|cselect|ff0|ff1|flbit|lshl|lshl1|lshl2|lshl3|lshl4|lshr|max|min|mov|movk|mul|mul_hi|mulk|nand|nor|not|"
    r"or|orn1|orn2|pack_ll|pack_lh|pack_hh|quadmask|sext|sub|subb|wqm|xnor|xor)"
    r"(_(eq|ne|lg|gt|ge|lt|le))?(_saveexec|_wrexec)?(_[iub]\d+)*")
CONTROL = re.compile(r"s_(barrier|branch|cbranch_(execn?z|vccn?z|scc[01])|endpgm|getpc_b64|setpc_b64|swappc_b64|nop|"
                     r"set_gpr_idx_(on|off|idx|mode)|setprio|sleep|waitcnt)")
PACKED_F32 = re.compile(r"v_pk_(add|mul|fma)_f32")


def allowed(mnemonic):
    return mnemonic in LOADS or ARITHMETIC.fullmatch(mnemonic) is not None or CONTROL.fullmatch(mnemonic) is not None


def _have_hipcc():
    try:
        B.hipcc()
        return True
    except RuntimeError:
        return False


def test_the_list():
    for m in ("s_load_dwordx4", "s_and_saveexec_b64", "s_cmp_lg_u64", "s_cmpk_lt_i32", "s_bcnt1_i32_b64", "s_mul_hi_u32",
              "s_cbranch_execz", "s_waitcnt", "s_ff1_i32_b64"):
        assert allowed(m), m
    for m in ("s_sendmsg", "s_trap", "s_icache_inv", "s_load_dwordx5", "s_memtime"):
        assert not allowed(m), m


@pytest.mark.skipif(not _have_hipcc(), reason="hipcc not available")
def test_scalar_instructions_only_read(tmp_path):
    def mnemonics(src):
        flags = [f for f in B.HIPCC_FLAGS if f != "-fPIC"]
        out = str(tmp_path / (src + ".s"))
        res = subprocess.run([B.hipcc(), *flags, "-I", B.INCLUDE, "-I", B.CSRC, "--cuda-device-only", "-S",
                              f"{B.CSRC}/{src}", "-o", out], capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-2000:]
        with open(out) as f:
            return set(re.findall(r"^\t(s_\w+|v_pk_\w+)", f.read(), flags=re.M))
    with ThreadPoolExecutor(max_workers=4) as ex:
        found = dict(zip(B.SOURCES, ex.map(mnemonics, B.SOURCES)))
    assert sum("s_load_dwordx2" in v for v in found.values()) > 5, "the kernels' assembly was not found"
    for src, names in found.items():
        bad = sorted(m for m in names if PACKED_F32.match(m) or (m.startswith("s_") and not allowed(m)))
        assert not bad, f"{src}: {bad}"

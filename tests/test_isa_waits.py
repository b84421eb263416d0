"""The built library holds no instruction that comes too early after one that
the hardware does not wait for (isa_waits.py states the rules), and the check
itself finds each kind in a made-up listing."""
import os
from collections import Counter

import pytest

import isa_waits
from paper_2609_32882_amd import build

LISTING = """
0000000000001000 <k>:
\ts_mov_b32 m0, s1                                           // 000000001000: BEFC0001
%s
\tglobal_load_lds_dwordx4 v1, s[4:5]                         // 000000001010: DDF48000 00040001
\tv_mfma_f32_32x32x16_bf16 a[0:15], v[2:5], v[6:9], a[0:15]  // 000000001018: D3B70000 00000000
\tv_mfma_f32_32x32x16_bf16 a[0:15], v[2:5], v[6:9], a[0:15]  // 000000001020: D3B70000 00000000
\ts_cbranch_scc1 65530                                       // 000000001028: BF85FFFA <k+0x%x>
%s
\tv_accvgpr_read_b32 v3, a7                                  // 000000001030: D3D84003 00000107
\ts_endpgm                                                   // 000000001038: BF810000
"""
NOP0 = "\ts_nop 0                                                    // 000000001004: BF800000"
NOP19 = "\ts_nop 15                                                   // 00000000102C: BF80000F\n" \
        "\ts_nop 2                                                    // 00000000102E: BF800002"
READLANE = "\tv_readlane_b32 s4, v9, s0                                  // 000000001008: D2890004 00000109"


@pytest.mark.parametrize("mid,back,tail,want", [
    (NOP0, 0x18, NOP19, {}),
    ("", 0x18, NOP19, {"m0": 1}),
    (READLANE, 0x18, NOP19, {"sgpr": 1}),
    (NOP0, 0x30, NOP19, {"acc": 2}),          # the branch skips the waits behind the products
    (NOP0, 0x18, "", {"acc": 2}),
])
def test_the_check_finds_missing_waits(mid, back, tail, want):
    found = isa_waits.violations(LISTING % (mid, back, tail))
    assert Counter(v.split(":")[0] for v in found) == want


def test_the_built_kernels_keep_their_waits(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    listings = isa_waits.disassemble(build.LIB, str(tmp_path))
    kernels = [isa_waits.parse(x) for x in listings]
    # the check reaches what it is about: copies into LDS and hand-written products
    assert sum(i.lds_load for k in kernels for c in k.values() for i in c) > 1000
    assert sum(bool(i.acc) for k in kernels for c in k.values() for i in c) > 100
    found = [v for x in listings for v in isa_waits.violations(x)]
    assert not found, "%d missing waits, first: %s" % (len(found), found[:3])


EXEC = """
0000000000001000 <k>:
%s
\ts_mov_b64 exec, 1                                          // 000000001004: BEFE0181
\tglobal_store_dword v1, v2, s[4:5]                          // 000000001008: DC708000 00040201
\ts_mov_b64 exec, %s                                         // 000000001010: BEFE0106
\ts_endpgm                                                   // 000000001014: BF810000
"""
KEPT = "\ts_mov_b64 s[6:7], exec                                     // 000000001000: BE86017E"


@pytest.mark.parametrize("first,back,found", [(KEPT, "s[6:7]", 0), (KEPT, "-1", 1), (KEPT, "s[8:9]", 1), (NOP0, "s[6:7]", 1)])
def test_the_check_finds_lanes_left_switched(first, back, found):
    assert len(isa_waits.exec_constants(isa_waits.parse(EXEC % (first, back))["k"])) == found


def test_the_built_kernels_put_their_lanes_back(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    codes = [c for x in isa_waits.disassemble(build.LIB, str(tmp_path)) for c in isa_waits.parse(x).values()]
    # the pacing words' stores: there are some
    assert sum(i.op == "s_mov_b64" and i.args == "exec, 1" for c in codes for i in c) > 0
    found = [v for c in codes for v in isa_waits.exec_constants(c)]
    assert not found, found[:3]

"""CPU-side checks of the C ABI: the library loads, exports every declared symbol, and its host
logic (budget rules, validation, error codes) behaves as include/thrift.h says.  No kernel runs."""
import ctypes as C
import os
import re

import pytest

from paper_2605_23081_amd import binding as T

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "thrift.h")).read()
    declared = set(re.findall(r"\b(thrift_[a-z0-9_]+)\s*\(", header))
    assert declared == set(T.EXPORTS), declared ^ set(T.EXPORTS)
    L = T.lib()
    for name in declared:
        assert hasattr(L, name), name


def test_host_budget_helpers_match_the_oracle(oracle):
    for vis in (0, 1, 19, 20, 21, 64, 2048):
        for f in (0.0, 1e-7, 0.01, 0.05, 0.1, 0.25, 0.999999, 1.0):
            assert T.row_budget(vis, f) == oracle.row_k(vis, f)
        assert T.row_budget(vis, 0.5, fixed_k=7) == oracle.row_k(vis, 0.5, 7)
    for Bq, Bk, Tk in ((64, 64, 32), (128, 64, 64), (1, 64, 16)):
        for i in range(0, 16):
            assert T.visible_blocks(i, Tk, Bq, Bk, True) == oracle.visible_blocks(i, Tk, Bq, Bk, True)
    assert T.visible_blocks(0, 2048, 1, 64, True, 131071) == 2048
    for n, f in ((32, 0.05), (512, 0.05), (2048, 0.25)):
        assert T.budget_to_global_k(n, f) == oracle.paper_global_k(n, f)
    assert T.select_kmax(32, 32, 64, 64, True, 0.05) == 2
    assert T.select_kmax(1024, 2048, 128, 64, True, 0.05) == 103
    assert T.select_kmax(8, 8, 64, 64, False, 0.0, fixed_k=3) == 3


def test_validation_errors_come_before_any_launch():
    L = T.lib()
    fake = C.c_void_p(0x1000)   # never dereferenced: every call below must fail validation first
    NULL, SHAPE, DTYPE, BUDGET, WORKSPACE = 1, 2, 3, 4, 5
    assert L.thrift_block_means(None, 0, 1, 1, 64, 128, 64, fake, None) == NULL
    assert L.thrift_block_means(fake, 0, 1, 1, 64, 64, 64, fake, None) == SHAPE      # D != 128
    assert L.thrift_block_means(fake, 0, 1, 1, 100, 128, 0, fake, None) == SHAPE     # block < 1
    assert L.thrift_block_means(fake, 0, 1, 1, 0, 128, 64, fake, None) == SHAPE      # empty sequence
    assert L.thrift_block_means(fake, 7, 1, 1, 64, 128, 64, fake, None) == DTYPE
    assert L.thrift_block_means(fake, 2, 1, 1, 64, 128, 64, fake, None) == DTYPE     # fp32 is output-only
    assert L.thrift_quantize_mxfp4(fake, 0, 1, 1, 0, 128, 1, fake, fake, None) == SHAPE    # empty sequence
    assert L.thrift_quantize_mxfp4(fake, 0, 1, 1, 64, 128, 2, fake, fake, None) == SHAPE
    sel = lambda **kw: L.thrift_select_topk(fake, fake, 1, kw.get("Hq", 4), kw.get("Hkv", 2), 8, kw.get("Tk", 8), 128, 64, 64, 1,
                                            C.c_double(kw.get("budget", 0.05)), kw.get("fixed_k", -1), 0, fake, fake,
                                            kw.get("kmax", 8), None)
    assert sel(Hq=3) == SHAPE
    assert sel(Tk=5000) == SHAPE
    assert sel(budget=1.5) == BUDGET
    assert sel(budget=-0.1) == BUDGET
    assert sel(budget=1.0, kmax=4) == BUDGET           # kmax too small for a 100 % budget
    pre = lambda **kw: L.thrift_attn_prefill(fake, fake, fake, kw.get("dt", 0), fake, fake, fake, fake, fake, fake, fake, fake, 4,
                                             1, 4, kw.get("Hkv", 2), kw.get("N", 256), kw.get("D", 128), kw.get("Bq", 64),
                                             kw.get("Bk", 64), 1, C.c_float(0.0), kw.get("out", fake), kw.get("odt", 0), None,
                                             None, 0, None)
    assert pre(Bq=32) == SHAPE and pre(Bk=128) == SHAPE and pre(D=64) == SHAPE and pre(N=0) == SHAPE and pre(Hkv=3) == SHAPE
    assert pre(out=None) == NULL
    assert pre(odt=5) == DTYPE and pre(dt=2) == DTYPE
    dec = lambda **kw: L.thrift_attn_decode(fake, 0, fake, fake, fake, fake, fake, fake, fake, None, 1, 4, 2, kw.get("N", 1024), 128, 64,
                                            C.c_double(kw.get("budget", 0.05)), -1, kw.get("split", 8), C.c_float(0.0), fake, 0,
                                            None, None, 0, kw.get("ws", fake), kw.get("wsb", 1 << 30), None)
    assert dec(split=0) == SHAPE and dec(N=1000) == SHAPE
    assert dec(budget=2.0) == BUDGET
    assert dec(ws=None) == WORKSPACE and dec(wsb=16) == WORKSPACE
    app = lambda **kw: L.thrift_kv_cache_append(kw.get("k", fake), fake, kw.get("dt", 0), kw.get("n", 1), kw.get("sl", fake), None,
                                                fake, fake, fake, fake, fake, fake, fake, 1, 2, kw.get("N", 1024), kw.get("D", 128),
                                                kw.get("Bk", 64), None)
    assert app(k=None) == NULL and app(sl=None) == NULL
    assert app(n=0) == SHAPE and app(n=2000) == SHAPE and app(N=1000) == SHAPE and app(D=64) == SHAPE and app(Bk=32) == SHAPE
    assert app(dt=2) == DTYPE
    fwd = lambda **kw: L.thrift_attention_forward(kw.get("q", fake), fake, fake, kw.get("dt", 1), 1, 4, kw.get("Hkv", 2), kw.get("N", 300),
                                                  kw.get("D", 128), kw.get("Bq", 128), 64, 1, C.c_double(kw.get("budget", 0.05)), -1, 0,
                                                  C.c_float(0.0), fake, 1, None, kw.get("ws", fake), kw.get("wsb", 16), None)
    assert fwd(q=None) == NULL and fwd(dt=2) == DTYPE and fwd(Hkv=3) == SHAPE and fwd(N=0) == SHAPE and fwd(Bq=32) == SHAPE
    assert fwd(budget=1.5) == BUDGET and fwd(ws=None) == WORKSPACE and fwd(wsb=16) == WORKSPACE
    # an unknown tile order is refused before the first stage of the chain is enqueued (it reaches only the last stage)
    assert L.thrift_attention_forward(fake, fake, fake, 1, 1, 4, 2, 300, 128, 128, 64, 1, C.c_double(0.05), -1, 7, C.c_float(0.0),
                                      fake, 1, None, fake, 1 << 30, None) == SHAPE
    # the entry point without a workspace argument: sizes are checked against its static array first
    sta = lambda **kw: L.thrift_attn_decode_static(fake, 0, fake, fake, fake, fake, fake, fake, fake, None, kw.get("B", 1), 4, 2,
                                                   kw.get("N", 1024), 128, 64, C.c_double(0.05), -1, kw.get("split", 8), C.c_float(0.0),
                                                   fake, 0, None, None, 0, None)
    assert sta(split=0) == SHAPE and sta(N=1000) == SHAPE
    assert sta(B=4096, N=131072, split=256) == WORKSPACE
    wsq = L.thrift_attention_forward_workspace
    assert wsq(1, 4, 2, 300, 128, 128, 64, 1, C.c_double(0.05), -1) > 300 * 128 * 6 // 2
    assert wsq(1, 4, 2, 300, 64, 128, 64, 1, C.c_double(0.05), -1) == 0 and wsq(1, 4, 2, 300, 128, 128, 64, 1, C.c_double(-1.0), -1) == 0
    need = T.decode_workspace_bytes(16, 32, 8, 131072, 128, 64, 256)
    assert 0 < need < (64 << 20)
    assert T.decode_workspace_bytes(16, 32, 8, 131072, 64, 64, 256) == 0
    assert "gfx950" in T.status_string(6)


def test_a_partition_of_the_whole_row_or_more_is_one_partition():
    """Sizes up to the largest int name the same problem as the row's own number of key blocks."""
    for Hq, Hkv, N in ((32, 8, 4096), (8, 8, 131072), (24, 2, 1024), (4, 4, 64)):
        need = T.decode_workspace_bytes(2, Hq, Hkv, N, 128, 64, N // 64)
        for split in (N // 64 + 1, 1 << 20, 2 ** 31 - N // 64, 2 ** 31 - 1):
            assert T.decode_workspace_bytes(2, Hq, Hkv, N, 128, 64, split) == need


def test_least_decode_workspace():
    """Never more than the workspace of the faster form; the same where there is no other form; 0 for what no form takes."""
    for B, Hq, Hkv, N, split in ((1, 32, 8, 131072, 256), (8, 64, 8, 32768, 256), (16, 32, 8, 131072, 256), (1, 4, 4, 64, 256), (2, 24, 2, 1024, 8)):
        need, least = (f(B, Hq, Hkv, N, 128, 64, split) for f in (T.decode_workspace_bytes, T.decode_least_workspace_bytes))
        assert 0 < least <= need
    assert T.decode_least_workspace_bytes(1, 32, 8, 131072, 128, 64, 256) < T.decode_workspace_bytes(1, 32, 8, 131072, 128, 64, 256)
    assert T.decode_least_workspace_bytes(16, 32, 8, 131072, 128, 64, 256) == T.decode_workspace_bytes(16, 32, 8, 131072, 128, 64, 256)
    assert T.decode_least_workspace_bytes(1, 32, 8, 100, 128, 64, 256) == 0


def test_peak_probe_validates_before_launching():
    L = T.lib()
    fake, work = C.c_void_p(0x1000), C.c_double(0.0)
    probe = lambda kind=4, dt=1, iters=10, buf=fake, size=1 << 30: L.thrift_peak_probe(kind, dt, iters, buf, C.c_size_t(size), C.byref(work), None)
    assert probe(buf=None) == 1
    assert probe(kind=5) == 2 and probe(kind=-1) == 2
    assert probe(iters=0) == 2
    assert probe(size=(16 << 20) - 1) == 2                 # smaller than the probes' result region
    assert probe(buf=C.c_void_p(0x1008)) == 2              # not 16-byte aligned
    assert probe(kind=1, dt=2) == 3                        # the 16-bit MFMA probe needs fp16 or bf16
    assert L.thrift_peak_probe(4, 1, 10, fake, C.c_size_t(1 << 30), None, None) == 1


def test_without_a_gpu_valid_calls_fail_loudly():
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    fake = C.c_void_p(0x1000)
    assert T.lib().thrift_block_means(fake, 0, 1, 1, 64, 128, 64, fake, None) == 6   # THRIFT_ERR_ARCH, nothing launched


def test_pre_pass_kernels_do_not_spill(tmp_path):
    """The selection keeps a row's keys in registers: up to 128 of them, next to the chains being scored."""
    import subprocess
    from paper_2605_23081_amd import build
    listing = tmp_path / "prepass.s"
    subprocess.run(["hipcc", *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, "thrift_prepass.hip"), "-o", str(listing)],
                   check=True, capture_output=True)
    assert build.scratch_in_loops(listing.read_text()) == []


def test_spill_check_reads_the_compiler_listing():
    """The build refuses a fused kernel whose listing touches scratch memory inside a loop (and only then)."""
    from paper_2605_23081_amd.build import scratch_in_loops
    listing = "\n".join([
        "_ZN6thrift4walkEv:",
        "; %bb.0:",
        "\tscratch_store_dword off, v1, off offset:16 ; 4-byte Folded Spill",          # before the loop: fine
        ".LBB0_1:                                ; =>This Inner Loop Header: Depth=1",
        "\tv_add_f32_e32 v0, v0, v1",
        "; %bb.2:                                ;   in Loop: Header=BB0_1 Depth=1",
        "\ts_cbranch_scc1 .LBB0_1",
        ".LBB0_3:",
        "\tscratch_load_dword v1, off, off offset:16 ; 4-byte Folded Reload",           # after it: fine
        "\ts_endpgm",
        "_ZN6thrift3badEv:",
        ".LBB1_1:                                ; =>This Inner Loop Header: Depth=1",
        "; %bb.2:                                ;   in Loop: Header=BB1_1 Depth=1",
        "\tscratch_load_dword v1, off, off ; 4-byte Folded Reload",
        "\ts_cbranch_scc1 .LBB1_1",
        "\ts_endpgm",
    ])
    assert scratch_in_loops(listing) == ["_ZN6thrift3badEv"]
    # a persistent kernel's outermost loop runs over work items: a reload at an item's start is outside the walk, one in
    # a nested loop (whose header line names the parent first and itself on the comment line below) is inside it
    def persistent(name, reload_in_walk):
        return "\n".join([
            name + ":",
            ".LBB2_1:                                ; =>This Loop Header: Depth=1",
            "\tscratch_load_dword v1, off, off offset:8 ; 4-byte Folded Reload",
            ".LBB2_2:                                ;   Parent Loop BB2_1 Depth=1",
            "                                        ; =>  This Inner Loop Header: Depth=2",
            "\tscratch_load_dword v2, off, off ; 4-byte Folded Reload" if reload_in_walk else "\tv_add_f32_e32 v0, v0, v1",
            "\ts_cbranch_scc1 .LBB2_2",
            "; %bb.3:                                ;   in Loop: Header=BB2_1 Depth=1",
            "\ts_cbranch_scc1 .LBB2_1",
            "\ts_endpgm",
        ])
    assert scratch_in_loops(persistent("_ZN6thrift17persistent_kernelEv", False)) == []
    assert scratch_in_loops(persistent("_ZN6thrift17persistent_kernelEv", True)) == ["_ZN6thrift17persistent_kernelEv"]
    assert scratch_in_loops(persistent("_ZN6thrift5otherEv", False)) == ["_ZN6thrift5otherEv"]


def test_listing_checks_refuse_a_format_they_cannot_read():
    """A listing without the labels the checks rely on must not pass for clean."""
    from paper_2605_23081_amd.build import m0_outside_inline_asm, scratch_in_loops
    for text in ("", "kernel_without_mangled_name:\n\tscratch_load_dword v1, off, off\n\ts_endpgm",
                 "_ZN6thrift4walkEv:\n\tv_add_f32_e32 v0, v0, v1\n\ts_endpgm"):          # no basic blocks, no loop annotation
        with pytest.raises(RuntimeError):
            scratch_in_loops(text)
    with pytest.raises(RuntimeError):
        m0_outside_inline_asm("\ts_mov_b32 m0, s10\n\tglobal_load_lds_dwordx4 v1, s[2:3]")   # no inline-assembly markers


def test_m0_check_reads_the_compiler_listing():
    from paper_2605_23081_amd.build import m0_outside_inline_asm
    ok = "\n".join(["\t;;#ASMSTART", "\ts_mov_b32 m0, s10", "\ts_nop 0", "\tglobal_load_lds_dwordx4 v1, s[2:3]", "\t;;#ASMEND",
                    "\tv_add_u32_e32 v0, v1, v2", "; a comment that mentions m0"])
    assert m0_outside_inline_asm(ok) == 0
    assert m0_outside_inline_asm(ok + "\n\ts_mov_b32 m0, -1\n\tds_gws_init v0 gds") == 1


def test_decode_workspace_holds_scores_for_two_launches_only():
    """What one launch keeps in LDS is not asked for where no budget takes two launches, so that the form fits wherever two launches
    with their scores would; and the form in finer pieces always asks for more than the walk, since the size of a workspace chooses
    between them."""
    size = lambda B, Hq, Hkv, Tk, split=256: T.decode_workspace_bytes(B, Hq, Hkv, 64 * Tk, 128, 64, split)
    scores = lambda B, Hq, Tk: B * Hq * Tk * 64 * 4
    for B, Hq, Hkv, Tk in ((3, 32, 8, 128), (1, 32, 8, 2048), (4, 64, 8, 512), (16, 32, 8, 128), (7, 8, 8, 2048)):
        assert size(B, Hq, Hkv, Tk) < scores(B, Hq, Tk)                      # one launch
    for B, Hq, Hkv, Tk in ((1, 32, 8, 1024), (1, 64, 8, 1024), (1, 32, 8, 129), (1, 32, 8, 64)):
        assert scores(B, Hq, Tk) < size(B, Hq, Hkv, Tk)                      # two
    for Hq, Hkv in ((1, 1), (16, 16), (16, 8), (32, 8), (64, 8), (7, 1)):
        for B in (1, 3, 16):
            for Tk in (1, 2, 63, 128, 129, 512, 1024):
                for split in (17, 256, 4096):
                    least = T.decode_least_workspace_bytes(B, Hq, Hkv, 64 * Tk, 128, 64, split)
                    if B * Hkv * -(-Tk // min(split, Tk)) <= 448:
                        assert size(B, Hq, Hkv, Tk, split) >= least + 256


def test_decode_takes_one_launch_where_it_is_the_faster_form():
    """Known by the scores in the workspace, which any budget's two launches ask for.  Four query heads per KV head just above 8192 key
    blocks are slower in one launch (53.1 us against 48.6 for 4 sequences of 264 blocks), eight up to 10240 (81.0 against 76.0 for one
    of 1280); without promoted blocks short rows of few blocks are (21.5 against 17.1 for 2 x 84 with four heads), one head up to 32768
    and eight heads in long rows (47.6 against 42.3 for 2 x 800)."""
    two = lambda B, Hq, Hkv, Tk: T.decode_workspace_bytes(B, Hq, Hkv, 64 * Tk, 128, 64, 256) > B * Hq * Tk * 64 * 4
    assert two(4, 32, 8, 264) and two(2, 32, 8, 576) and two(2, 16, 8, 576) and two(1, 16, 16, 576)
    assert not two(1, 32, 8, 1153) and not two(5, 16, 8, 257) and not two(1, 16, 16, 2049)
    assert two(2, 64, 8, 576) and two(1, 64, 8, 1280) and two(2, 40, 8, 640)
    assert two(2, 32, 8, 84) and two(1, 64, 8, 128) and two(2, 32, 8, 96) and two(4, 16, 16, 128) and two(16, 16, 16, 128) and two(2, 64, 8, 800)
    assert not two(2, 32, 8, 97) and not two(4, 64, 8, 64) and not two(1, 64, 8, 1601)
    assert not two(16, 32, 8, 128) and not two(16, 64, 8, 64)                # short rows of many blocks


_listings, _compiler_output = {}, {}


def _listing(source, path):
    import subprocess
    from paper_2605_23081_amd import build
    if source not in _listings:
        done = subprocess.run(["hipcc", *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", str(path)], check=True, capture_output=True, text=True)
        _listings[source], _compiler_output[source] = path.read_text(), done.stderr
    return _listings[source]


@pytest.mark.parametrize("source", ["thrift_prefill_split.hip", "thrift_prefill.hip"])
def test_hand_written_instructions_wait_for_matrix_results(tmp_path, source):
    """The factors of a raised maximum multiply the accumulators that a matrix instruction before them may still be writing."""
    from paper_2605_23081_amd.build import matrix_results_read_early
    assert matrix_results_read_early(_listing(source, tmp_path / "listing.s")) == []


@pytest.mark.parametrize("source", ["thrift_prefill_split.hip", "thrift_prefill.hip", "thrift_decode.hip", "thrift_decode_split.hip"])
def test_hand_written_instructions_stay_clear_of_scalar_results(tmp_path, source):
    """A comparison and the choice by its result need two wait states between them, which nobody inserts inside an asm statement."""
    from paper_2605_23081_amd.build import scalars_read_early
    assert scalars_read_early(_listing(source, tmp_path / "listing.s")) == []


def test_the_key_mask_waits_for_the_scores(tmp_path):
    """Right behind the matrix instructions, with nothing between them that happens to take the time."""
    from paper_2605_23081_amd.build import matrix_results_read_early, scalars_read_early
    source = tmp_path / "mask.hip"
    source.write_text("""#include "thrift_tile.h"
using namespace thrift;
__global__ void mask_kernel(const v8h* a, const v8h* b, float* out, int n_valid) {
  const int lane = threadIdx.x & 63;
  v16f s[2];
  for (int t = 0; t < 2; ++t) {
    v16f zero = {0.f};
    s[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[64 * t + lane], b[lane], zero, 0, 0, 0);
  }
  mask_scores(s, lane >> 5, n_valid);
  for (int i = 0; i < 32; ++i) out[64 * i + lane] = s[i / 16][i % 16];
  asm volatile("; end");
}
""")
    listing = _listing(str(source), tmp_path / "listing.s")
    assert matrix_results_read_early(listing) == []
    if "v_cmp" in listing:                                   # (a mask without comparisons has no scalar results)
        assert scalars_read_early(listing) == []


def test_scalar_wait_state_check_reads_the_compiler_listing():
    from paper_2605_23081_amd.build import scalars_read_early

    def kernel(write, read, *between, by_hand=(True, True)):
        lines = ["_ZN6thrift4walkEv:", "; %bb.0:", "\tv_readfirstlane_b32 s90, v9"]
        for text, hand in ((write, by_hand[0]), (between, False), (read, by_hand[1])):
            text = list(text) if isinstance(text, tuple) else ["\t" + text]
            lines += ["\t;;#ASMSTART", *text, "\t;;#ASMEND"] if hand else text
        return "\n".join(lines + ["\ts_endpgm"])

    mask, compare = "v_cndmask_b32 v1, v2, v1, vcc", "v_cmp_lt_i32 vcc, 3, v4"
    found = [("_ZN6thrift4walkEv", mask)]
    for hands, expected in (((True, True), found), ((False, True), found), ((True, False), found), ((False, False), [])):
        assert scalars_read_early(kernel(compare, mask, by_hand=hands)) == expected
        assert scalars_read_early(kernel(compare, mask, "\ts_nop 0", by_hand=hands)) == expected
        assert scalars_read_early(kernel(compare, mask, "\ts_nop 1", by_hand=hands)) == []
    assert scalars_read_early(kernel(compare, mask, "\tv_add_f32_e32 v9, v9, v9", "\tv_add_f32_e32 v9, v9, v9")) == []
    assert scalars_read_early(kernel(compare, mask.replace("vcc", "s[2:3]"))) == []
    assert scalars_read_early(kernel("v_cmp_lt_i32 s[2:3], 3, v4", "v_add_f32 v1, s3, v1")) == [("_ZN6thrift4walkEv", "v_add_f32 v1, s3, v1")]
    assert scalars_read_early(kernel("v_add_co_u32 v1, vcc, v2, v3", "v_addc_co_u32 v4, s[4:5], v5, v6, vcc"))
    assert scalars_read_early(kernel("v_add_co_u32 v1, s[4:5], v2, v3", "v_add_co_u32 v4, s[4:5], v5, v6")) == []          # written, not read
    load = "global_load_lds_dword v1, s[2:3]"
    assert scalars_read_early(kernel("v_readfirstlane_b32 s3, v4", load, "\ts_nop 3", by_hand=(False, True)))
    assert scalars_read_early(kernel("v_readfirstlane_b32 s3, v4", load, "\ts_nop 4", by_hand=(False, True))) == []
    assert scalars_read_early(kernel("v_readfirstlane_b32 s3, v4", load, "\ts_add_i32 s3, s3, 1", by_hand=(False, True))) == []
    assert scalars_read_early(kernel("v_readfirstlane_b32 s3, v4", load, "\ts_cmp_eq_u32 s3, 1", by_hand=(False, True)))
    lane = "v_readlane_b32 s5, v4, s3"
    assert scalars_read_early(kernel("v_readfirstlane_b32 s3, v4", lane, "\ts_nop 2", by_hand=(False, True)))
    assert scalars_read_early(kernel("v_readfirstlane_b32 s3, v4", lane, "\ts_nop 3", by_hand=(False, True))) == []
    around = ["\ts_cbranch_scc1 .LBB0_2", "; %bb.1:", "\ts_nop 15", ".LBB0_2:"]
    assert scalars_read_early(kernel(compare, mask, "\ts_nop 0", *around)) == []
    assert scalars_read_early(kernel(compare, mask, *around)) == found
    with pytest.raises(RuntimeError):
        scalars_read_early("_ZN6thrift4walkEv:\n; %bb.0:\n\ts_endpgm")


def test_launch_bounds_are_met(tmp_path):
    """The compiler drops a bound that it cannot meet, and allocates registers as if there were none."""
    import subprocess
    from paper_2605_23081_amd import build
    for source in ("thrift_prefill.hip", "thrift_decode_split.hip"):
        _listing(source, tmp_path / "listing.s")
        assert build.unmet_launch_bounds(_compiler_output[source]) == []
    source = tmp_path / "bounds.hip"
    for waves_per_simd, unmet in ((2, []), (6, ["_Z13bounds_kernelPf"])):    # workgroups of two wavefronts whose LDS lets a CU hold three
        source.write_text("""#include <hip/hip_runtime.h>
__global__ void __launch_bounds__(128, %d) bounds_kernel(float* x) {
  __shared__ float lds[12544];
  lds[threadIdx.x] = x[threadIdx.x];
  __syncthreads();
  x[threadIdx.x] = lds[127 - threadIdx.x];
}
""" % waves_per_simd)
        done = subprocess.run(["hipcc", *build.FLAGS, "-S", "--cuda-device-only", str(source), "-o", str(tmp_path / "bounds.s")],
                              check=True, capture_output=True, text=True)
        assert build.unmet_launch_bounds(done.stderr) == unmet


def test_only_the_kernels_that_take_turns_set_a_priority(tmp_path):
    """The question whether a grid takes turns is the launch's, not one of every key block; every walk takes them where it is asked to."""
    text = _listing("thrift_prefill.hip", tmp_path / "listing.s")
    bodies = {name: body for name, body in re.findall(r"^(_ZN6thrift14prefill_kernel\w+):(.*?)^\.Lfunc_end", text, re.M | re.S)}
    assert len(bodies) == 28
    for name, body in bodies.items():
        assert ("s_setprio" in body) == name.endswith("ELi1EEEvNS_11PrefillArgsE"), name


def test_wait_state_check_reads_the_compiler_listing():
    from paper_2605_23081_amd.build import matrix_results_read_early

    def kernel(*between, op="v_mfma_scale_f32_32x32x64_f8f6f4 v[0:15], v[16:19], v[20:23], v[0:15], v24, v25 cbsz:4 blgp:4", read="v_mul_f32 v15, v30, v15"):
        return "\n".join(["_ZN6thrift4walkEv:", "; %bb.0:", "\t" + op, *between, "\t;;#ASMSTART", "\t" + read, "\t;;#ASMEND", "\ts_endpgm"])

    found = [("_ZN6thrift4walkEv", "v_mul_f32 v15, v30, v15")]
    assert matrix_results_read_early(kernel("\ts_nop 10")) == found
    assert matrix_results_read_early(kernel("\ts_nop 11")) == []
    assert matrix_results_read_early(kernel("\ts_nop 9", "\tv_add_f32_e32 v40, v41, v42 ; a comment")) == found
    assert matrix_results_read_early(kernel(read="v_mul_f32 v16, v30, v16")) == []                       # an operand, not the result
    small = "v_mfma_f32_16x16x32_f16 a[4:7], v[16:19], v[20:23], 0"
    assert matrix_results_read_early(kernel("\ts_nop 6", op=small, read="v_add_f32 v1, a7, v2")) == [("_ZN6thrift4walkEv", "v_add_f32 v1, a7, v2")]
    assert matrix_results_read_early(kernel("\ts_nop 7", op=small, read="v_add_f32 v1, a7, v2")) == []
    # two ways to the statement: past the wait, and around it; and once more around a loop
    around = ["\ts_cbranch_scc1 .LBB0_2", "; %bb.1:", "\ts_nop 15", ".LBB0_2:"]
    assert matrix_results_read_early(kernel(*around)) == found
    past = ["\ts_branch .LBB0_3", ".LBB0_2:", "\ts_endpgm", ".LBB0_3:", "\ts_nop 9"]
    assert matrix_results_read_early(kernel(*past)) == found
    assert matrix_results_read_early(kernel(*past, "\ts_nop 0")) == []
    loop = "\n".join(["_ZN6thrift4walkEv:", ".LBB0_1:", "\t;;#ASMSTART", "\tv_mul_f32 v3, v30, v3", "\t;;#ASMEND",
                      "\tv_mfma_f32_32x32x16_f16 v[0:15], v[16:19], v[20:23], v[0:15]", "\ts_cbranch_scc1 .LBB0_1", "\ts_endpgm"])
    assert matrix_results_read_early(loop) == [("_ZN6thrift4walkEv", "v_mul_f32 v3, v30, v3")]
    for text in ("", kernel().replace("\t;;#ASMSTART\n", ""), kernel(op="v_add_f32_e32 v0, v1, v2")):
        with pytest.raises(RuntimeError):
            matrix_results_read_early(text)

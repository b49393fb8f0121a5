"""What the compiler makes of the kernels, read without a GPU.  The GEMM kernels must not spill: a spill in the K loop would go
unnoticed at run time, and its reload would wait for the tile loads that the kernel counts by itself.  The kernel file is compiled to
gfx950 assembly, or the built library's notes are read, for the resource usage that the compiler reports per kernel."""
import os
import re
import struct
import subprocess
import tempfile

from paper_2006_09503_amd import build as B

from gpu_util import GEMM_TILE_FORMS


def test_ring_gemm_kernels_use_no_scratch_and_fit_two_waves_per_simd():
    src = os.path.join(B.CSRC, "gemm_bf16.hip")
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "gemm_bf16.s")
        flags = [f for f in B.FLAGS if f != "-fPIC"]
        subprocess.run([B.HIPCC, *flags, "--cuda-device-only", "-S", src, "-o", out], check=True,
                       stderr=subprocess.DEVNULL)
        text = open(out).read()
    kernels = re.findall(r"\.name:\s+(\S+)\n(.*?)\.wavefront_size", text, flags=re.S)
    ring = [(n, body) for n, body in kernels if "gemm_bf16_ring_kernel" in n]
    assert len(ring) >= 10
    for name, body in ring:
        field = lambda k: int(re.search(r"\." + k + r":\s+(\d+)", body).group(1))
        assert field("private_segment_fixed_size") == 0, name       # no scratch: nothing spilled
        assert field("vgpr_spill_count") == 0 and field("sgpr_spill_count") == 0, name
        assert field("vgpr_count") <= 256, name                     # 8 waves per workgroup = 2 per SIMD


def test_no_asm_load_leaves_a_register_in_flight():
    """The compiler takes the output of an asm block as written when the block ends.  A load whose register is written later may
    therefore only be issued by a block that waits for it as well."""
    blocks = []
    for name in sorted(os.listdir(B.CSRC)):
        if name.endswith((".hip", ".hpp", ".h")):
            text = open(os.path.join(B.CSRC, name)).read()
            blocks += [(name, b) for b in re.findall(r"\basm\s+(?:volatile\s*)?\((.*?)\);", text, flags=re.S)]
    assert any("global_load_lds" in b for _, b in blocks)      # the search finds the blocks there are
    for name, b in blocks:
        code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', b.split("\n")[0]))
        loads = re.search(r"\b(?:global|buffer|flat|scratch|ds|s)_(?:load|read|buffer_load)\w*", code)
        if loads and "_lds" not in loads.group(0):
            assert "s_waitcnt" in code, (name, b)


def test_phased_gemm_kernels_do_not_spill():
    kernels = built_kernels("gemm_bf16_phased_kernel")
    assert len(kernels) >= 10
    for name, field in kernels:
        assert field("private_segment_fixed_size") == 0 and field("vgpr_spill_count") == 0 and field("sgpr_spill_count") == 0, name
        assert field("vgpr_count") <= 256, name                     # 8 waves per workgroup = 2 per SIMD


def built_kernels(pattern):
    """(demangled name, field reader) of the kernels whose name holds `pattern` in the library as it is built, from the notes of its
    gfx950 code objects."""
    llvm = os.path.join(os.path.dirname(os.path.dirname(B.HIPCC)), "llvm", "bin")
    if not os.path.exists(B.LIB):
        B.build()
    data, out, at = open(B.LIB, "rb").read(), [], 0
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    with tempfile.TemporaryDirectory() as tmp:
        while (at := data.find(magic, at)) >= 0:
            n, p = struct.unpack_from("<Q", data, at + len(magic))[0], at + len(magic) + 8
            for _ in range(n):
                offset, size, length = struct.unpack_from("<QQQ", data, p)
                target, p = data[p + 24:p + 24 + length], p + 24 + length
                if b"gfx950" not in target or size == 0:
                    continue
                path = os.path.join(tmp, "code.o")
                with open(path, "wb") as f:
                    f.write(data[at + offset:at + offset + size])
                out.append(subprocess.run([os.path.join(llvm, "llvm-readelf"), "--notes", path], check=True, capture_output=True,
                                          text=True).stdout)
            at += len(magic)
    kernels = re.findall(r"\.name:\s+(\S+)\n(.*?)\.wavefront_size", "\n".join(out), flags=re.S)
    names = subprocess.run(["c++filt"], input="\n".join(n for n, _ in kernels), capture_output=True, text=True).stdout.split("\n")
    return [(name, lambda k, body=body: int(re.search(r"\." + k + r":\s+(\d+)", body).group(1)))
            for name, (_, body) in zip(names, kernels) if re.search(pattern, name)]


def test_small_head_attention_kernels_leave_room_for_two_workgroups_per_cu():
    """256-row workgroups are 8 waves; with at most 128 registers a CU holds two.  A dQ kernel of 141 cost the backward pass at head
    size 32 up to a quarter of its speed."""
    for kernel, head in (("fwd", 32), ("fwd", 64), ("dq", 32), ("dkv", 32), ("bwd", 32)):
        found = built_kernels(rf"attn_{kernel}_mfma_kernel<{head}, 8, 1, false")
        assert found, (kernel, head)
        for name, field in found:
            assert field("vgpr_count") <= 128 and field("private_segment_fixed_size") == 0, name


def test_fixed_head_attention_kernels_do_not_spill():
    """The instances of head sizes 32, 64, 80 and 128 (those of the padded sizes hold a second, row-by-row copy of their loop, which
    spills).  Two registers in front of the loop of the 64-row dQ kernel at head size 128 are the exception, and four of the kernel that
    holds the whole backward pass of such blocks."""
    found = built_kernels(r"attn_(fwd|dq|dkv|bwd)_mfma_kernel<\d+, \d, \d, false")
    assert len(found) >= 45
    allowed = {"attn_dq_mfma_kernel<128, 4, 2": 2, "attn_bwd_mfma_kernel<128, 4, 2": 4}
    for name, field in found:
        assert field("vgpr_spill_count") <= sum(n for kernel, n in allowed.items() if kernel in name), name


def test_every_operand_form_has_the_tile_variants_that_the_tests_force():
    """A forced variant that a form has not gives way to the built-in choice without a word: what the tests take for granted is what is
    built."""
    shapes = {"gemm_bf16_kernel<128, 128, 64, 64, 64, {}, 1>": 2, "gemm_bf16_kernel<256, 256, 128, 64, 64, {}, 1>": 3,
              "gemm_bf16_kernel<128, 128, 64, 64, 64, {}, 2>": 6, "gemm_bf16_ring_kernel<128, 128, 32, 64, 64, 4, {}>": 22,
              "gemm_bf16_ring_kernel<256, 256, 128, 64, 32, 4, {}>": 23, "gemm_bf16_ring_kernel<192, 256, 96, 64, 32, 4, {}>": 24,
              "gemm_bf16_phased_kernel<256, 256, 128, 64, {}>": 25, "gemm_bf16_phased_kernel<192, 256, 96, 64, {}>": 26,
              "gemm_bf16_phased_kernel<128, 256, 64, 64, {}>": 27, "gemm_bf16_split_kernel<1, 1, 8, {}>": 32,
              "gemm_bf16_split_kernel<2, 2, 4, {}>": 64}
    forms = {"f": [("false, false, %d" % e) for e in (0, 1, 2)], "d": [("false, true, %d" % e) for e in (0, 2)], "w": ["true, false, 3"]}
    expected = {pattern.format(args) for pattern, tile in shapes.items() for form in GEMM_TILE_FORMS[tile] for args in forms[form]}
    built = {re.search(r"gemm_bf16\w*<[^>]*>", name).group(0) for name, _ in built_kernels(r"gemm_bf16\w*<")}
    assert built == expected, built ^ expected


def test_fp32_attention_kernels_do_not_spill():
    """Their rare second run, for infinities and NaNs that some rows must not see, works on 32 columns of the results at a time; with all at
    once 92 to 302 registers spilled at head sizes 48, 64, 112 and 128, some in the loop of the first run.  Six of the second run at head
    size 64, dQ and dK/dV in one launch, are the exception."""
    found = built_kernels(r"attn_f32_(fwd|dq|dkv|bwd)_kernel<")
    assert len(found) == 64
    for name, field in found:
        assert field("vgpr_spill_count") <= (6 if "attn_f32_bwd_kernel<64" in name else 0), name


def test_phased_gemm_kernels_use_no_scratch_and_fit_two_waves_per_simd():
    """They park the next-weights touch in a register as the ring kernels do."""
    found = built_kernels(r"gemm_bf16_phased_kernel<")
    assert len(found) >= 10
    for name, field in found:
        assert field("private_segment_fixed_size") == 0 and field("vgpr_spill_count") == 0 and field("sgpr_spill_count") == 0, name
        assert field("vgpr_count") <= 256, name


def test_narrow_fp32_gemm_kernels_have_one_instance_per_form_and_do_not_spill():
    """16 x 16 tiles: one number of chunks in flight at every K (a second instance for long K was slower than 32 x 32 tiles from K = 257 to
    about 450, and than the first one everywhere)."""
    found = built_kernels(r"gemm_f32_narrow_kernel<")
    assert {re.search(r"<([^>]*)>", name).group(1) for name, _ in found} == {f"{tb}, {epi}" for tb in ("false", "true") for epi in range(4)}
    for name, field in found:
        assert field("private_segment_fixed_size") == 0 and field("vgpr_spill_count") == 0 and field("sgpr_spill_count") == 0, name


def test_folded_fp32_attention_backward_does_not_spill_in_its_loops():
    """The causal backward launch in the folded order, of the head sizes of which a CU holds two workgroups: as its plain form, it spills at head
    size 64 only, four registers of the rare second run, and has a few bytes of scratch at 32."""
    found = built_kernels(r"attn_f32_bwd_folded_kernel<")
    assert sorted(int(re.search(r"<(\d+)>", name).group(1)) for name, _ in found) == [16, 32, 48, 64]
    for name, field in found:
        assert field("vgpr_spill_count") <= (4 if "<64>" in name else 0), name
        assert field("private_segment_fixed_size") <= {"<64>": 44, "<32>": 36}.get(re.search(r"<\d+>", name).group(0), 0), name


def test_fp32_gemm_kernels_that_hold_a_layernorm_or_the_sums_do_not_spill():
    found = built_kernels(r"gemm_f32_(ln|wgrad_sums)_kernel")
    assert len(found) == 13      # forward (plain, GELU) and backward (plain, GELU') of 1, 2 and 4 chunks; the weight gradients
    for name, field in found:
        assert field("private_segment_fixed_size") == 0 and field("vgpr_spill_count") == 0 and field("sgpr_spill_count") == 0, name

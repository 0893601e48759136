"""What the compiler made of a few lines the kernels depend on (CPU: hipcc cross-compiles gfx950 to assembly)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_19849_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"


def _assembly(src, tmp_path):
    out = tmp_path / (src + ".s")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-S", "--cuda-device-only", "-o", str(out), os.path.join(CSRC, src)],
                   check=True, stderr=subprocess.DEVNULL)
    return out.read_text()


def _kernel_body(asm, mangled):
    start = asm.index("\n" + mangled + ":")
    end = asm.index(".end_amdhsa_kernel", start)
    return asm[start:end]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_combine_keeps_cached_and_streaming_loads_apart(tmp_path):
    """The combine kernel reads just-dispatched rows with cached loads and all others with streaming (nt) loads,
    in two loops that differ in nothing else; an optimiser that folds them drops the hint (seen: all loads
    became cached ones, combine 98 -> 111 us).  Both kinds must be there, as many of one as of the other."""
    asm = _assembly("combine.hip", tmp_path)
    for mangled in ("_ZN2ep14combine_kernelILi1ELi8EEEvNS_11CombineArgsE",
                    "_ZN2ep14combine_kernelILi1ELi2EEEvNS_11CombineArgsE"):
        loads = re.findall(r"global_load_dwordx4[^\n]*", _kernel_body(asm, mangled))
        nt = [l for l in loads if re.search(r"\bnt\b", l)]
        assert len(nt) > 0 and len(nt) * 2 == len(loads), (mangled, len(nt), len(loads))


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_rows_are_counted_behind_their_reservation(tmp_path):
    """One command per row: an expert's rows are counted (the add at an address of the lane's own) once the reservation of
    their Idx has returned.  The wait stands in the source, for nothing else orders two relaxed adds."""
    asm = _assembly("dispatch.hip", tmp_path)
    kernels = re.findall(r"^(_ZN2ep\d+dispatch_(?:bf16|fp8)_kernelILi\d+ELb1E\w*):", asm, re.M)
    assert len(kernels) == 10
    for mangled in kernels:
        body = _kernel_body(asm, mangled)
        counted = list(re.finditer(r"global_atomic_add v\d+, v\[\d+:\d+\], v\d+, off sc0", body))
        assert len(counted) == 1, mangled
        reserved = body.rindex("global_atomic_add_x2", 0, counted[0].start())
        assert re.search(r"#ASMSTART\s+s_waitcnt vmcnt\(0\)\s+;+#ASMEND", body[reserved:counted[0].start()]), mangled


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_fp8_form_for_one_rank_has_one_copy_of_the_row_loads(tmp_path):
    """A dispatch to one rank of several reads every token's pairs first and few rows: a kernel without the row loads ahead of
    the pairs, which cost it scalar registers though it never takes them."""
    asm = _assembly("dispatch.hip", tmp_path)
    kernels = re.findall(r"^(_ZN2ep19dispatch_fp8_kernelILi(\d+)ELb0ELb0ELb0E\w*):", asm, re.M)
    assert len(kernels) == 3
    for mangled, vpl in kernels:
        body = _kernel_body(asm, mangled)
        assert len(re.findall(r"global_load_dwordx4 [^\n]*\bnt\b", body)) == 2 * int(vpl), mangled
        assert int(re.search(r"\.amdhsa_next_free_sgpr (\d+)", asm[asm.index(".amdhsa_kernel " + mangled):])[1]) <= 96, mangled


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_rows_of_tokens_without_experts_are_not_read_ahead(tmp_path):
    """A kernel that reads rows ahead of the tokens' pairs, and not in small launches only, asks for the first pair before: a
    scalar load of the expert, and what comes of its sign.  Tokens that name none (padding) cost no read of their row."""
    asm = _assembly("dispatch.hip", tmp_path)
    kernels = re.findall(r"^(_ZN2ep20dispatch_bf16_kernelILi\d+ELb0ELi2E\w*|_ZN2ep19dispatch_fp8_kernelILi\d+ELb0ELb1E\w*):",
                         asm, re.M)
    assert len(kernels) == 3 + 6
    for mangled in kernels:
        body = _kernel_body(asm, mangled)
        first_row = re.search(r"global_load_dwordx4 [^\n]*\bnt\b", body).start()
        assert re.search(r"s_load_dword (s\d+), s\[\d+:\d+\], 0x0\s+s_waitcnt lgkmcnt\(0\)\s+s_cmp_gt_i32 \1, -1\b",
                         body[:first_row]), mangled


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_ring_kernel_waits_for_its_invalidate(tmp_path):
    """One wave drops the stale lines for its whole workgroup.  The barrier behind it orders the other waves' loads only if
    the invalidate is through by then: the wave waits for a load of its own behind it."""
    body = _kernel_body(_assembly("ht_ring.hip", tmp_path), "_ZN2ep14ht_ring_kernelENS_10HtRingArgsE")
    behind = [m.end() for m in re.finditer(r"\bbuffer_inv sc1\b", body)]
    assert behind
    for at in behind:
        to_barrier = body[at:body.index("s_barrier", at)]
        assert re.search(r"global_load_dword v\d+, [^\n]*\n(?:[^\n]*\n)*?\s*s_waitcnt vmcnt\(0\)", to_barrier), to_barrier


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_ring_kernel_passes_over_groups_that_a_narrow_row_does_not_have(tmp_path):
    """A lane's eight groups of channels are quantised one behind the other; ahead of each stands a branch of the whole wave,
    for rows that end before it."""
    body = _kernel_body(_assembly("ht_ring.hip", tmp_path), "_ZN2ep14ht_ring_kernelENS_10HtRingArgsE")
    converted = [m.start() for m in re.finditer(r"\bv_cvt_pk_fp8_f32\b", body)]
    assert len(converted) == 8 * 8
    for i in range(8, 64, 8):
        assert re.search(r"\bs_cbranch_(?:scc|vcc)", body[converted[i - 1]:converted[i]]), i // 8


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_ring_kernel_with_another_first_argument_is_refused(tmp_path):
    """The ring kernel reads its channels' state at an offset from the start of the argument block, so nothing may come to
    stand before the one argument it has."""
    def compiles(src):
        f = tmp_path / "ht_ring.hip"
        f.write_text(src)
        r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only", "-I" + CSRC, str(f)],
                           capture_output=True, text=True)
        return r.returncode == 0, r.stderr

    with open(os.path.join(CSRC, "ht_ring.hip")) as f:
        src = f.read()
    ok, err = compiles(src)
    assert ok, err
    moved = src.replace("ht_ring_kernel(HtRingArgs a)", "ht_ring_kernel(int first, HtRingArgs a)").replace(
        "(hipStream_t)stream, b)", "(hipStream_t)stream, 0, b)")
    ok, err = compiles(moved)
    assert not ok and err.count("error: ") and "ht_fifo" in err, err

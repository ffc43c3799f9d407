"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol that
include/still.h declares, and rejects bad arguments before anything is launched."""
import ctypes
import os
import re

import pytest

from paper_2602_02180_amd import binding as S

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "still.h")).read()
    return sorted(set(re.findall(r"STILL_API\s+[\w\s\*]+?\b(still_\w+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = declared_symbols()
    assert {"still_hybrid_attn_fwd", "still_hybrid_attn_decode_step", "still_fwd_workspace_bytes",
            "still_state_bytes", "still_state_init", "still_last_error", "still_version",
            "still_hybrid_attn_decode_step_at", "still_hybrid_attn_fwd_static", "still_hybrid_attn_bwd",
            "still_bwd_workspace_bytes", "still_bwd_workspace_layout", "still_attention_map",
            "still_attention_map_bwd", "still_attention_map_bwd_workspace_bytes", "still_rope_apply"} <= set(names)
    lib = S.lib()
    for n in names:
        assert hasattr(lib, n), n
    assert S.still_version() >= 100


def params(**kw):
    base = dict(B=1, N=1024, Hq=4, Hkv=2, d=64, C=64, W=64, lam=16, scale=0.125, eps=1e-6, dtype="bf16")
    base.update(kw)
    return S.make_params(**base)


def test_workspace_layout_is_consistent():
    p = params()
    L = S.still_fwd_workspace_layout(p)
    assert S.still_fwd_workspace_bytes(p) == L.total
    offs = [L.score, L.sel, L.vt, L.kret, L.vrett, L.wqt, L.wkf, L.seg, L.snap, L.zsnap, L.pimg, L.zpre, L.kmask, L.n_la, L.d_la, L.vfr, L.ev_src, L.ev_alive, L.ev_fin, L.ev_vfr, L.lse, L.total]
    assert offs == sorted(offs) and all(o % 256 == 0 for o in offs)
    assert L.n_pad % 128 == 0 and L.n_pad >= 1024
    assert L.cap % 64 == 0 and L.cap >= (1024 // 64) * 16
    assert L.nseg * L.seg_chunks >= 16
    assert L.snap - L.seg >= 1 * 4 * L.nseg * (2 * 64 * 65) * 4
    assert L.zsnap - L.snap >= 1 * 4 * 16 * 64 * 128 * 2           # one bf16 state per (head, chunk)
    assert L.zpre - L.pimg >= 1 * 4 * L.nseg * 64 * 128 * 2        # and one per (head, segment)
    assert L.d_la - L.n_la <= 256                                   # the inspection regions are empty by default
    Lt = S.still_fwd_workspace_layout(params(emit_terms=1))
    assert Lt.d_la - Lt.n_la >= 1 * 4 * 1024 * 64 * 4 and Lt.total > L.total


def test_retained_budget_bounds_the_retained_rows_of_workspace_and_state():
    free = S.still_fwd_workspace_layout(params(N=8192))
    tight = S.still_fwd_workspace_layout(params(N=8192, max_retained=100))
    assert free.cap == (8192 // 64) * 16 and tight.cap == 128
    assert tight.total < free.total
    roomy = S.still_fwd_workspace_layout(params(N=8192, max_retained=1 << 20))
    assert roomy.cap == free.cap and roomy.total == free.total
    # a decode state no longer grows with the context once the budget is set
    s_free = S.still_state_layout(params(N=1, max_tokens=1 << 20))
    s_tight = S.still_state_layout(params(N=1, max_tokens=1 << 20, max_retained=896))
    assert s_free.cap >= (1 << 20) // 64 * 16 and s_tight.cap == 896 + 64
    assert s_tight.kret < s_tight.vret and s_tight.vret - s_tight.kret == 1 * 4 * s_tight.cap * 64 * 2


def test_eviction_policy_layouts():
    """Budget policy 1: the workspace holds ALL offers (the sparse kernel walks them under masks) plus the plan's
    regions; the decode state holds max_retained rows plus their scores and token indices."""
    stop = S.still_fwd_workspace_layout(params(N=8192, max_retained=100))
    ev = S.still_fwd_workspace_layout(params(N=8192, max_retained=100, budget_policy=1))
    assert stop.cap == 128 and ev.cap == (8192 // 64) * 16
    assert stop.ev_alive - stop.ev_src <= 256 and stop.lse - stop.ev_vfr <= 256      # empty without the policy
    assert ev.ev_alive - ev.ev_src >= 1 * 4 * 8192 * 4
    assert ev.ev_fin - ev.ev_alive >= 1 * 4 * (8192 // 64) * (ev.cap // 64) * 8
    assert ev.ev_vfr - ev.ev_fin >= 1 * 4 * (2 * 100 + 1) * 4
    assert ev.lse - ev.ev_vfr >= 1 * 4 * 64 * ev.n_pad * 2 and ev.total - ev.lse >= 1 * 4 * 8192 * 4
    s_stop = S.still_state_layout(params(N=1, max_tokens=1 << 20, max_retained=896))
    s_ev = S.still_state_layout(params(N=1, max_tokens=1 << 20, max_retained=896, budget_policy=1))
    assert s_ev.cap == s_stop.cap == 896 + 64
    assert s_stop.ret_tok - s_stop.ret_score <= 256
    assert s_ev.ret_tok - s_ev.ret_score >= 1 * 4 * s_ev.cap * 4 and s_ev.total - s_ev.ret_tok >= 1 * 4 * s_ev.cap * 4


@pytest.mark.parametrize("kw,code", [
    (dict(d=96), S.STILL_ERR_UNSUPPORTED),
    (dict(C=32), S.STILL_ERR_UNSUPPORTED),
    (dict(W=257, C=128), S.STILL_ERR_UNSUPPORTED),
    (dict(d_f=32), S.STILL_ERR_UNSUPPORTED),
    (dict(lam=65), S.STILL_ERR_INVALID_ARG),
    (dict(lam=-1), S.STILL_ERR_INVALID_ARG),
    (dict(N=0), S.STILL_ERR_INVALID_ARG),
    (dict(Hq=5), S.STILL_ERR_INVALID_ARG),
    (dict(eps=0.0), S.STILL_ERR_INVALID_ARG),
    (dict(kv_head_of_q=[0, 1, 2, 0]), S.STILL_ERR_INVALID_ARG),
    (dict(budget_policy=2, max_retained=64), S.STILL_ERR_INVALID_ARG),
    (dict(budget_policy=1), S.STILL_ERR_INVALID_ARG),                       # eviction needs a budget to hold
    (dict(budget_policy=1, max_retained=64, shared_selection=1), S.STILL_ERR_UNSUPPORTED),
    (dict(budget_policy=1, max_retained=5000), S.STILL_ERR_UNSUPPORTED),    # the retained set is ranked in LDS
])
def test_bad_params_are_rejected_on_the_host(kw, code):
    p = params(**kw)
    with pytest.raises(S.StillError) as e:
        S.still_fwd_workspace_layout(p)
    assert e.value.code == code
    assert S.still_last_error() != ""


def test_backward_entry_point_validates_on_the_host():
    """The backward pass covers budget_policy 0 without padding; fp32 only at d = 64; its workspace holds a forward
    workspace plus its own regions; null pointers are refused before any launch."""
    for kw in (dict(dtype="f32", d=128, C=128), dict(max_retained=64, budget_policy=1)):
        with pytest.raises(S.StillError) as e:
            S.still_bwd_workspace_layout(params(**kw))
        assert e.value.code == S.STILL_ERR_UNSUPPORTED
    p = params()
    BL = S.still_bwd_workspace_layout(p)
    assert S.still_bwd_workspace_bytes(p) == BL.total
    names = [n for n, t in S.StillBwdWsLayout._fields_ if t is ctypes.c_size_t]
    offs = [getattr(BL, n) for n in names]
    assert offs == sorted(offs) and all(o % 256 == 0 for o in offs)
    assert BL.e_row - BL.fwd >= S.still_fwd_workspace_bytes(p)
    assert BL.dz - BL.ds >= 1 * 4 * 16 * 128 * 64 * 2 and BL.total - BL.dv32 >= 1 * 2 * 1024 * 64 * 4
    p.q_st = p.k_st = p.v_st = p.o_st = 64
    null, fake = ctypes.c_void_p(None), ctypes.c_void_p(0x1000)
    rc = S.lib().still_hybrid_attn_bwd(ctypes.byref(p), fake, fake, fake, null, fake, null, fake, null, fake, fake,
                                        null, fake, fake, fake, fake, null, fake, null, fake, null, fake, 1 << 40, null)
    assert rc == S.STILL_ERR_INVALID_ARG and "pointer" in S.still_last_error()
    rc = S.lib().still_hybrid_attn_bwd(ctypes.byref(p), fake, fake, fake, null, fake, null, fake, null, fake, fake,
                                        fake, fake, fake, fake, fake, null, fake, null, fake, null, fake, 16, null)
    assert rc == S.STILL_ERR_WORKSPACE_TOO_SMALL
    rc = S.lib().still_hybrid_attn_bwd(ctypes.byref(p), fake, fake, fake, fake, fake, null, fake, null, fake, fake,
                                        fake, fake, fake, fake, fake, null, fake, null, fake, null, fake, 1 << 40, null)
    assert rc == S.STILL_ERR_INVALID_ARG and "dg" in S.still_last_error()


def test_rope_entry_point_validates_on_the_host():
    lib = S.lib()
    null, fake = ctypes.c_void_p(None), ctypes.c_void_p(0x1000)
    p = params()
    p.q_st = p.k_st = 64
    assert lib.still_rope_apply(ctypes.byref(p), null, null, null, ctypes.c_float(10000.0), null) == S.STILL_ERR_INVALID_ARG
    assert lib.still_rope_apply(ctypes.byref(p), fake, fake, null, ctypes.c_float(1.0), null) == S.STILL_ERR_INVALID_ARG
    assert "base" in S.still_last_error()
    p.q_st = 32
    assert lib.still_rope_apply(ctypes.byref(p), fake, null, null, ctypes.c_float(10000.0), null) == S.STILL_ERR_INVALID_ARG


def test_fwd_rejects_null_and_misaligned_pointers_without_launching():
    p = params()
    lib = S.lib()
    null = ctypes.c_void_p(None)
    rc = lib.still_hybrid_attn_fwd(ctypes.byref(p), null, null, null, null, null, null, null, null, null, null,
                                   null, 0, null, null, 0, null)
    assert rc == S.STILL_ERR_INVALID_ARG
    fake = ctypes.c_void_p(0x1000)
    odd = ctypes.c_void_p(0x1004)
    p.q_st = p.k_st = p.v_st = p.o_st = 64
    rc = lib.still_hybrid_attn_fwd(ctypes.byref(p), odd, fake, fake, null, fake, null, fake, null, fake, null,
                                   null, 0, null, fake, 1 << 40, null)
    assert rc == S.STILL_ERR_INVALID_ARG and "aligned" in S.still_last_error()
    p.q_st = 63   # not a multiple of 16 bytes
    rc = lib.still_hybrid_attn_fwd(ctypes.byref(p), fake, fake, fake, null, fake, null, fake, null, fake, null,
                                   null, 0, null, fake, 1 << 40, null)
    assert rc == S.STILL_ERR_INVALID_ARG
    p = params()
    p.q_st = p.k_st = p.v_st = p.o_st = 64
    rc = lib.still_hybrid_attn_fwd(ctypes.byref(p), fake, fake, fake, null, fake, null, fake, null, fake, null,
                                   null, 0, null, fake, 16, null)
    assert rc == S.STILL_ERR_WORKSPACE_TOO_SMALL


def test_state_export_with_injected_indices_needs_scores_and_is_rejected_before_any_launch():
    """state_out carries the scores of the local span; with injected indices the scores are only computed when
    score_out is given.  The combination without score_out is refused by the host checks (fake pointers: a launch
    would fault), as the header promises for every failure."""
    p = params(max_tokens=1024)
    p.q_st = p.k_st = p.v_st = p.o_st = 64
    lib = S.lib()
    null, fake = ctypes.c_void_p(None), ctypes.c_void_p(0x1000)
    rc = lib.still_hybrid_attn_fwd(ctypes.byref(p), fake, fake, fake, null, fake, null, fake, null, fake, null,
                                   fake, 1, fake, fake, 1 << 40, null)
    assert rc == S.STILL_ERR_INVALID_ARG and "score" in S.still_last_error()


def test_side_entry_points_validate_only_what_they_read():
    """The global score and the overlap count do not touch the linear branch: its restrictions (d_f == d, W <= 256,
    no fp32 with d = C = 128) must not be applied to them.  Null pointers make the calls stop right after the
    parameter checks, with the pointer message."""
    lib = S.lib()
    null = ctypes.c_void_p(None)
    for kw in (dict(dtype="f32", d=128, C=128), dict(d_f=32), dict(W=4096), dict(C=32, lam=0)):
        p = params(**kw)
        p.q_st = p.k_st = kw.get("d", 64)
        rc = lib.still_global_score(ctypes.byref(p), null, null, null, null)
        assert rc == S.STILL_ERR_INVALID_ARG and "pointer" in S.still_last_error(), (kw, S.still_last_error())
    p = params(C=32, lam=7, d_f=5, W=999)
    rc = lib.still_selection_overlap(ctypes.byref(p), null, null, null, null)
    assert rc == S.STILL_ERR_INVALID_ARG and "pointer" in S.still_last_error()
    for kw, code in ((dict(d=96), S.STILL_ERR_UNSUPPORTED), (dict(eps=0.0), S.STILL_ERR_INVALID_ARG)):
        p = params(**kw)
        assert lib.still_global_score(ctypes.byref(p), null, null, null, null) == code
    for kw, code in ((dict(C=256), S.STILL_ERR_UNSUPPORTED), (dict(lam=65), S.STILL_ERR_INVALID_ARG)):
        p = params(**kw)
        assert lib.still_selection_overlap(ctypes.byref(p), null, null, null, null) == code


def test_public_header_is_plain_c_and_matches_the_binding(tmp_path):
    """include/still.h compiles as C99 on its own, and the struct sizes the C compiler sees are the ones the ctypes
    binding marshals (a field added on one side only would shift every later field)."""
    import shutil
    import subprocess

    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no C compiler")
    src = tmp_path / "sizes.c"
    src.write_text('#include <stdio.h>\n#include <stddef.h>\n#include "still.h"\n'
                   'int main(void) { printf("%zu %zu %zu %zu %zu\\n", sizeof(still_params_t), sizeof(still_ws_layout_t),\n'
                   '  sizeof(still_state_layout_t), offsetof(still_params_t, q_sb), offsetof(still_params_t, seq_len));\n'
                   '  return 0; }\n')
    exe = tmp_path / "sizes"
    subprocess.run([gcc, "-std=c99", "-Wall", "-Wextra", "-Werror", "-pedantic", "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe)], check=True)
    got = [int(x) for x in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]
    assert got == [ctypes.sizeof(S.StillParams), ctypes.sizeof(S.StillWsLayout), ctypes.sizeof(S.StillStateLayout),
                   S.StillParams.q_sb.offset, S.StillParams.seq_len.offset]


@pytest.mark.parametrize("kw", [
    dict(B=5, N=768, Hq=26, Hkv=2, lam=8), dict(B=2, N=768, Hq=66, Hkv=1, lam=4), dict(B=6, N=763, Hq=22, Hkv=2, lam=4),
    dict(B=2, N=768, Hq=72, Hkv=6, lam=0), dict(B=7, N=512, Hq=37, Hkv=1, lam=0)], ids=lambda k: f"{k['B']}x{k['N']}x{k['Hq']}")
def test_the_cut_of_the_scan_never_outgrows_the_builtin_scratch_array(kw):
    """Problems that fit the built-in scratch array only when the scan is cut into few segments keep the few.  That the
    cheapest cut is another one shows with emit_terms, which takes more than the array either way: more segments, and
    that many more would not have fitted."""
    kw = dict(kw, d=64, C=128)
    few, cheap = S.still_fwd_workspace_layout(params(**kw)), S.still_fwd_workspace_layout(params(emit_terms=1, **kw))
    assert few.total <= 32 << 20 < cheap.total
    assert few.seg_chunks > cheap.seg_chunks and few.nseg < cheap.nseg
    per_segment = kw["B"] * kw["Hq"] * (2 * 64 * 65 * 4 + 64 * 2 * 64 * 2 + 2 * 64 * 4)   # totals, image and z of one segment
    assert few.total + (cheap.nseg - few.nseg) * per_segment > 32 << 20


def test_the_backward_workspace_holds_what_the_kernels_use_and_no_more():
    """The training shape (16 sequences of 1024 tokens, 32 / 8 heads, d = 128, C = 64, bf16): the forward workspace, per query
    head and token three scalars, A, phi of either side, df of either side and a fp32 row, the state gradients, per kv head and
    token two fp32 rows, per retained entry (64 more than the lists hold) two rows, two fp32 rows, four bytes and a bit,
    and two copies of the weights; every region is rounded up to 256 bytes."""
    B, N, Hq, Hkv, d, C, lam = 16, 1024, 32, 8, 128, 64, 16
    p = params(B=B, N=N, Hq=Hq, Hkv=Hkv, d=d, C=C, W=128, lam=lam)
    rows, entries = B * Hq * N, B * Hq * (N // C * lam + 64)
    want = S.still_fwd_workspace_bytes(p) + rows * (12 + 2 * d + 2 * 4 * d + 2 * 2 * d + 4 * d) \
        + B * Hq * (N // C) * 2 * d * (2 * d + 4) + 2 * 4 * B * Hkv * N * d + entries * (2 * 2 * d + 2 * 4 * d + 4) \
        + entries // 8 + 4 * Hq * d * d
    assert want <= S.still_bwd_workspace_bytes(p) <= want + 64 * 256
    assert S.still_attention_map_bwd_workspace_bytes(p) <= S.still_bwd_workspace_bytes(p) + 4 * rows + 256


def test_the_backward_pass_reads_no_retained_row_behind_its_buffers(tmp_path):
    """The key side of the linear branch reads, for every chunk that has retained entries, rows from the chunk's first to the last
    slot that counts, whether a token is retained or not.  Under a budget the buffers stop growing with the chunks: the
    rows of every chunk, by the kernel's own rule, lie inside what the workspace layout gives a head."""
    import random
    import subprocess

    from paper_2602_02180_amd import build

    src, exe = tmp_path / "rows.hip", tmp_path / "rows"
    src.write_text('#include <cstdio>\n#include "still_kernels.h"\n'
                   'int main() {\n  int nc, lam, n_ret;\n'
                   '  while (std::scanf("%d %d %d", &nc, &lam, &n_ret) == 3) {\n    int last = -1;\n'
                   '    for (int c = 0; c + 2 < nc; ++c) {\n      if (still::retained_row(c, lam, 0, n_ret) < 0) continue;\n'
                   '      for (int pos = 0; pos < lam; ++pos) {\n        const int row = still::retained_row(c, lam, pos, n_ret);\n'
                   '        last = row > last ? row : last;\n      }\n    }\n    std::printf("%d\\n", last);\n  }\n  return 0;\n}\n')
    subprocess.run([build.HIPCC, "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-w",
                    "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    rng, calls = random.Random(5), []
    for _ in range(400):
        kw = dict(B=rng.randint(1, 3), Hq=rng.choice([1, 4, 8]), d=rng.choice([64, 128]), C=rng.choice([64, 128]),
                  N=rng.randint(1, 32768), max_retained=rng.choice([0, 1, 5, 64, 128, 200, 896, rng.randint(1, 4000)]))
        kw.update(Hkv=1, lam=rng.choice([1, 7, 16, 32, kw["C"]]))
        nc = -(-kw["N"] // kw["C"])
        n_ret = max(0, nc - 2) * kw["lam"]
        if kw["max_retained"]:
            n_ret = min(n_ret, kw["max_retained"])
        calls.append((kw, nc, n_ret))
    text = "".join(f"{nc} {kw['lam']} {n_ret}\n" for kw, nc, n_ret in calls)
    out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True).stdout.split()
    short = 0
    for (kw, nc, n_ret), last in zip(calls, map(int, out)):
        L = S.still_bwd_workspace_layout(params(**kw))
        assert last == n_ret - 1 and last < max(L.cap_t, 1), (kw, last)
        assert L.dvret - L.dkret >= kw["B"] * kw["Hq"] * L.cap_t * kw["d"] * 4
        short += (nc - 3) * kw["lam"] >= L.cap_t       # the first row of the last such chunk would lie behind the buffer
    assert short > 50


def test_the_state_scan_spills_no_addresses(tmp_path):
    """Registers of every instance of the scan, as the compiler reports them: its image store must not hold an address per entry
    (in fp32 at d = 128, whose accumulators alone fill the register file, that was 2458 spilled values and a kernel
    1.8 times as slow)."""
    import subprocess

    from paper_2602_02180_amd import build

    run = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-c", os.path.join(build.CSRC, "still_la.hip"), "-o",
                          str(tmp_path / "la.o"), "-Rpass-analysis=kernel-resource-usage"], check=True, capture_output=True, text=True)
    found = re.findall(r"Function Name: (\S*la_kernel\S*)(?:.|\n)*?VGPRs Spill: (\d+)", run.stderr)
    spills = {name: int(n) for name, n in found}
    assert len(spills) == 16
    for name, n in spills.items():
        assert n <= (460 if "la_kernelIfLi128" in name else 0), (name, n)

"""Host-side checks of the C ABI: the library loads, exports every symbol that
include/flmoe.h declares, and its host-only entry points validate arguments.
No kernel is launched here."""
import ctypes as C
import math
import os
import re
import subprocess
import sys

import pytest

from paper_2510_27656_amd import flmoe

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "flmoe.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(fl_moe_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = declared_symbols()
    assert "fl_moe_layout" in names and "fl_moe_combine_reduce" in names and len(names) >= 12
    L = flmoe.lib()
    for n in names:
        assert hasattr(L, n), n
    assert sorted(flmoe.EXPORTS) == names


def cfg(**kw):
    base = dict(n_ranks=32, n_experts=256, max_tokens=128, top_k=8, hidden=7168,
                dispatch_dtype=0, expert_align=1, flags=0, recv_capacity_rows=0,
                expert_capacity_rows=0, spin_limit=0)
    base.update(kw)
    return flmoe.fl_moe_config(**base)


def test_query_sizes_decode_shape():
    s = flmoe.fl_moe_query_sizes(cfg())
    assert s.x_row_bytes == 14336 and s.wire_row_bytes == 14336 and s.combine_row_bytes == 14336
    assert s.recv_capacity_rows == 32 * 128
    assert s.expert_capacity_rows == 32 * 128 * 8
    assert s.send_capacity_rows == 128 * 8
    assert s.workspace_bytes % 256 == 0
    # the two receive buffers dominate: every pair's reply, every received row
    payload = 32 * (1024 * 14336 + 4096 * 14336)
    assert payload <= s.workspace_bytes <= 1.05 * payload
    s8 = flmoe.fl_moe_query_sizes(cfg(dispatch_dtype=1))
    assert s8.wire_row_bytes == 7424 and s8.scales_per_row == 56      # 7168 + 4*56 = 7392, on 128-byte lines
    assert s8.expert_x_row_bytes == 7168
    payload = 32 * (1024 * 14336 + 4096 * 7424)
    assert payload <= s8.workspace_bytes <= 1.05 * payload


def test_capacities_are_clamped_and_padding_counted():
    s = flmoe.fl_moe_query_sizes(cfg(expert_align=16, expert_capacity_rows=0))
    assert s.expert_capacity_rows == 32 * 128 * 8 + 7 * 15
    s = flmoe.fl_moe_query_sizes(cfg(recv_capacity_rows=10 ** 9, expert_capacity_rows=2000))
    assert s.recv_capacity_rows == 32 * 128 and s.expert_capacity_rows == 2000


def test_private_rows_extend_the_receive_buffer():
    base = flmoe.fl_moe_query_sizes(cfg())
    assert base.private_rows == 0 and base.recv_buffer_rows == base.recv_capacity_rows
    s = flmoe.fl_moe_query_sizes(cfg(max_private_rows=32))
    assert s.private_rows == 32
    assert s.recv_buffer_rows == 32 * 32 + s.recv_capacity_rows
    assert s.workspace_bytes > base.workspace_bytes
    # a source never sends more than T rows to one destination
    s = flmoe.fl_moe_query_sizes(cfg(max_private_rows=10 ** 6))
    assert s.private_rows == 128
    # the shared range can then be configured smaller
    s = flmoe.fl_moe_query_sizes(cfg(max_private_rows=32, recv_capacity_rows=1024))
    assert s.recv_buffer_rows == 32 * 32 + 1024


@pytest.mark.parametrize("bad,code", [
    (dict(n_ranks=0), flmoe.FL_ERR_INVALID_ARG),
    (dict(n_ranks=65, n_experts=65), flmoe.FL_ERR_INVALID_ARG),
    (dict(n_experts=250), flmoe.FL_ERR_INVALID_ARG),
    (dict(top_k=17), flmoe.FL_ERR_INVALID_ARG),
    (dict(top_k=0), flmoe.FL_ERR_INVALID_ARG),
    (dict(hidden=100), flmoe.FL_ERR_ALIGNMENT),
    (dict(hidden=(1 << 20) + 8), flmoe.FL_ERR_INVALID_ARG),
    (dict(hidden=192, dispatch_dtype=1), flmoe.FL_ERR_ALIGNMENT),
    (dict(dispatch_dtype=7), flmoe.FL_ERR_INVALID_ARG),
    (dict(expert_align=0), flmoe.FL_ERR_INVALID_ARG),
    (dict(flags=32), flmoe.FL_ERR_INVALID_ARG),
    (dict(flags=flmoe.FL_FLAG_STREAM_ORDERED | flmoe.FL_FLAG_PROGRESSIVE_RECV), flmoe.FL_ERR_INVALID_ARG),
    (dict(max_tokens=0), flmoe.FL_ERR_INVALID_ARG),
    (dict(max_private_rows=-1), flmoe.FL_ERR_INVALID_ARG),
    (dict(reserved=1), flmoe.FL_ERR_INVALID_ARG),
])
def test_query_sizes_rejects_bad_configs(bad, code):
    with pytest.raises(flmoe.FlMoeError) as ei:
        flmoe.fl_moe_query_sizes(cfg(**bad))
    assert ei.value.code == code


def test_null_arguments_are_errors_not_crashes():
    L = flmoe.lib()
    assert L.fl_moe_query_sizes(None, None) == flmoe.FL_ERR_INVALID_ARG
    assert L.fl_moe_destroy(None) == flmoe.FL_ERR_INVALID_ARG
    assert L.fl_moe_layout(None, 0, 1, None, None, None, None) == flmoe.FL_ERR_INVALID_ARG
    assert L.fl_moe_dispatch_send(None, 0, 1, None, None) == flmoe.FL_ERR_INVALID_ARG
    assert L.fl_moe_status(None, None, None) == flmoe.FL_ERR_INVALID_ARG
    assert L.fl_moe_required_capacities(None, None, None, None) == flmoe.FL_ERR_INVALID_ARG
    assert L.fl_moe_strerror(flmoe.FL_ERR_WORKSPACE) == b"workspace too small"
    names = [L.fl_moe_kernel_name(i).decode() for i in range(flmoe.FL_KERNEL_COUNT)]
    assert all(names) and len(set(names)) == flmoe.FL_KERNEL_COUNT


def test_large_calls_are_cut_into_rank_groups_small_ones_are_not():
    """Host rule behind the launches of a payload call: one launch while the ranks of the
    call move at most three times the per-launch target (860 MiB by default), otherwise
    groups of ranks of about the target size; row = the larger of wire and combine row."""
    groups = flmoe.fl_moe_debug_launch_groups
    dsv3 = dict(n_ranks=32, n_experts=256, top_k=8, hidden=7168)
    per_rank_128 = 128 * 8 * 14336
    assert per_rank_128 * 32 <= 3 * (860 << 20)
    assert groups(cfg(max_tokens=128, **dsv3), 32) == 32          # decode: 470 MB, one launch
    assert groups(cfg(max_tokens=512, **dsv3), 32) == 32          # 1.9 GB: still one launch
    assert groups(cfg(max_tokens=1024, **dsv3), 32) == 7          # 3.8 GB -> 5 launches
    assert groups(cfg(max_tokens=2048, **dsv3), 32) == 4
    assert groups(cfg(max_tokens=4096, **dsv3), 32) == 2          # prefill: 16 launches of 2 ranks
    assert groups(cfg(max_tokens=4096, **dsv3), 1) == 1           # one real rank's call is never cut
    assert groups(cfg(max_tokens=4096, **dsv3), 32, 0) == 32      # knob 0: never cut
    assert groups(cfg(max_tokens=128, **dsv3), 32, 1) == 1        # tiny target: one rank per launch
    assert groups(cfg(max_tokens=1 << 20, **dsv3), 32) == 1       # never below one rank
    assert groups(cfg(max_tokens=4096, flags=flmoe.FL_FLAG_STREAM_ORDERED, **dsv3), 32) == 2
    assert groups(cfg(max_tokens=4096, flags=flmoe.FL_FLAG_PROGRESSIVE_RECV, **dsv3), 32) == 32   # polling receivers: never cut
    # e4m3 dispatch: the combine row (bf16) is the larger one and decides
    assert groups(cfg(max_tokens=4096, dispatch_dtype=flmoe.FL_DTYPE_E4M3_BLOCK128, **dsv3), 32) == 2
    lib = flmoe.lib()
    out = C.c_int(0)
    c = cfg(max_tokens=128, **dsv3)
    assert lib.fl_moe_debug_launch_groups(C.byref(c), 0, -1, C.byref(out)) == flmoe.FL_ERR_INVALID_ARG
    assert lib.fl_moe_debug_launch_groups(C.byref(c), 33, -1, C.byref(out)) == flmoe.FL_ERR_INVALID_ARG
    assert lib.fl_moe_debug_launch_groups(C.byref(c), 32, -1, None) == flmoe.FL_ERR_INVALID_ARG


# (change to 16 ranks x 8 experts, 1024 tokens, 128-byte rows; unpack, replies by chunks of rows?)
@pytest.mark.parametrize("kw,unpack,replies", [
    (dict(), 1, 1),
    (dict(max_tokens=16), 0, 0),                       # rows fit on the machine as one wave each
    (dict(max_tokens=40), 0, 0),                       # 5 120 replies: as many as there are waves
    (dict(max_tokens=41), 0, 1),
    (dict(hidden=1024), 1, 1),
    (dict(hidden=1032), 0, 0),                         # rows of more than 2 KB
    (dict(hidden=2048, dispatch_dtype=1), 1, 0),       # 2 KB of codes, replies of 4 KB
    (dict(flags=flmoe.FL_FLAG_PARTIAL_SUMS, hidden=768), 1, 1),
    (dict(flags=flmoe.FL_FLAG_PARTIAL_SUMS, hidden=776), 1, 0),
    (dict(flags=flmoe.FL_FLAG_PROGRESSIVE_RECV, hidden=7168, max_tokens=1), 1, 1),
    (dict(recv_capacity_rows=300, expert_capacity_rows=300), 0, 0),
])
def test_many_short_rows_are_moved_by_chunks(kw, unpack, replies):
    """Waves on their own start and end at a bounded rate: 16 ranks of 4096 tokens with 128-byte rows took 689 us a
    step by waves and 222 by chunks.  Longer rows, and few rows, go by waves."""
    c = dict(n_ranks=16, n_experts=128, max_tokens=1024, top_k=8, hidden=64)
    c.update(kw)
    plan = flmoe.fl_moe_debug_launch_plan(cfg(**c), 16)
    assert (plan.unpack_by_chunks, plan.replies_by_chunks) == (unpack, replies)
    single = flmoe.fl_moe_debug_launch_plan(cfg(**dict(c, max_tokens=40)), 1)      # a rank by itself has few rows
    if not c.get("flags", 0) & flmoe.FL_FLAG_PROGRESSIVE_RECV:
        assert (single.unpack_by_chunks, single.replies_by_chunks) == (0, 0)
    with pytest.raises(flmoe.FlMoeError):
        flmoe.fl_moe_debug_launch_plan(cfg(**c), 17)


@pytest.mark.parametrize("N,El,K,T", [(8, 1, 8, 1024), (16, 1, 8, 4096), (8, 2, 8, 4096), (2, 2, 3, 500), (32, 8, 8, 128),
                                      (1, 16, 4, 77), (4, 1, 1, 64), (64, 16, 16, 300)])
def test_grids_cover_the_mean_and_six_deviations_of_uniform_routing(N, El, K, T):
    """A token's experts are distinct, so with few experts per rank it reaches more ranks than K independent draws
    would: it misses a rank in C(E - El, K) of C(E, K) choices."""
    E = N * El
    for flags in (0, flmoe.FL_FLAG_PARTIAL_SUMS):
        plan = flmoe.fl_moe_debug_launch_plan(cfg(n_ranks=N, n_experts=E, max_tokens=T, top_k=K, hidden=4096,
                                                  flags=flags), N)
        hit = 1 - math.comb(E - El, K) / math.comb(E, K)
        mean, room = N * T * hit, N * T                      # a rank never receives more than every token
        assert plan.recv_grid_rows >= min(room, mean + 6 * math.sqrt(N * T * hit * (1 - hit)))
        assert plan.recv_grid_rows <= min(room, mean + 6 * math.sqrt(mean) + 3)
        if flags:
            assert plan.reply_grid_rows == plan.recv_grid_rows
        else:
            assert min(N * T * min(K, El), T * K + 6 * math.sqrt(T * K)) <= plan.reply_grid_rows <= T * K + 6 * math.sqrt(T * K) + 3


def test_replies_are_cached_by_the_size_of_the_whole_group():
    """Rank by rank, 1.75 GiB of replies took 2794 us a step through the caches and 2704 past them: what decides is
    what all ranks write before the first reduce, not what one call writes."""
    dsv3 = dict(n_ranks=32, n_experts=256, top_k=8, hidden=7168)
    cached = lambda tokens, ranks: flmoe.fl_moe_debug_launch_plan(cfg(max_tokens=tokens, **dsv3), ranks).replies_cached
    assert cached(128, 32) and cached(128, 16) and cached(128, 1)      # 448 MiB
    assert cached(256, 32) and not cached(256, 1)                      # 896 MiB
    assert not cached(512, 32) and not cached(512, 16) and not cached(512, 1)


# ranks x tokens of 7168 values, top 8, one rank a call: 320 workgroups and many, replies of 35 MiB to 1.75 GiB
@pytest.mark.parametrize("N,T", [(32, 128), (32, 147), (32, 160), (32, 256), (32, 465), (64, 128), (16, 320), (16, 400), (8, 700),
                                 (4, 16), (32, 512)])
@pytest.mark.parametrize("flags", [0, flmoe.FL_FLAG_PARTIAL_SUMS, flmoe.FL_FLAG_ZERO_PAD])
def test_a_reply_kernel_that_streams_never_announces(N, T, flags):
    """Streamed replies are in memory when their kernel ends, not when its workgroups have seen them acknowledged."""
    for hidden in (7168, 64, 1 << 20):
        c = cfg(n_ranks=N, n_experts=8 * N, max_tokens=T if hidden < 1 << 20 else 2, hidden=hidden, flags=flags)
        for ranks in {1, 2, N // 2, N}:
            for cached_mb in (-1, 0, 1, 64, 1 << 20):
                plan = flmoe.fl_moe_debug_ordering_plan(c, ranks, cached_mb)
                assert plan.replies_written_through or plan.combine_announce_kernel, (hidden, ranks, cached_mb)


def test_which_calls_announce_with_a_kernel():
    plan = lambda ranks=32, mb=-1, **kw: flmoe.fl_moe_debug_ordering_plan(cfg(**kw), ranks, mb)
    small, large = plan(max_tokens=4), plan(max_tokens=128)
    assert (small.dispatch_announce_kernel, small.replies_written_through, small.combine_announce_kernel) == (0, 1, 0)
    assert (large.dispatch_announce_kernel, large.replies_written_through, large.combine_announce_kernel) == (1, 1, 1)
    apart = plan(ranks=1, max_tokens=256)                   # few workgroups a call, 896 MiB of replies in the group
    assert (apart.replies_written_through, apart.combine_announce_kernel) == (1, 0)
    for streamed in (plan(ranks=1, max_tokens=512), plan(max_tokens=4, mb=0)):
        assert (streamed.replies_written_through, streamed.combine_announce_kernel) == (0, 1)
    for flag in (flmoe.FL_FLAG_STREAM_ORDERED, flmoe.FL_FLAG_PROGRESSIVE_RECV):
        own = plan(max_tokens=512, flags=flag)
        assert (own.dispatch_announce_kernel, own.combine_announce_kernel) == (0, 0)
        assert own.replies_written_through == (flag == flmoe.FL_FLAG_PROGRESSIVE_RECV)
    lib, out = flmoe.lib(), flmoe.fl_moe_ordering_plan()
    for ranks, mb in ((0, -1), (33, -1), (32, -2)):
        assert lib.fl_moe_debug_ordering_plan(C.byref(cfg()), ranks, mb, C.byref(out)) == flmoe.FL_ERR_INVALID_ARG
    assert lib.fl_moe_debug_ordering_plan(C.byref(cfg()), 32, -1, None) == flmoe.FL_ERR_INVALID_ARG


def test_which_calls_wait_behind_a_gate_kernel():
    """Receive launches of up to 1024 waves wait themselves: 32 ranks x 1 token of 14 waves each, not 2; 8 rows of a rank."""
    gates = lambda ranks, **kw: (lambda p: (p.dispatch_gate_kernel, p.combine_gate_kernel))(
        flmoe.fl_moe_debug_ordering_plan(cfg(**kw), ranks))
    tiny = dict(n_ranks=2, n_experts=8, max_tokens=16, top_k=2, hidden=256)
    assert gates(2, **tiny) == (0, 0) and gates(32, max_tokens=4) == (1, 1) and gates(1, max_tokens=4) == (0, 0)
    assert gates(32, max_tokens=1)[1] == 0 and gates(32, max_tokens=2)[1] == 1
    assert gates(1, max_tokens=4096) == (1, 1)
    for flag in (flmoe.FL_FLAG_STREAM_ORDERED, flmoe.FL_FLAG_PROGRESSIVE_RECV):
        assert gates(32, max_tokens=128, flags=flag) == (0, 0)


@pytest.mark.parametrize("hidden,dtype,dispatch,combine", [
    (7168, flmoe.FL_DTYPE_BF16, 14336, 14336), (7176, flmoe.FL_DTYPE_BF16, 14464, 14464), (1016, flmoe.FL_DTYPE_BF16, 2048, 2048),
    (520, flmoe.FL_DTYPE_BF16, 1040, 1040), (8, flmoe.FL_DTYPE_BF16, 16, 16), (7168, flmoe.FL_DTYPE_E4M3_BLOCK128, 7424, 14336)])
def test_row_strides_of_the_receive_buffers(hidden, dtype, dispatch, combine):
    """Rows start on 128-byte lines where that takes at most a sixteenth more room, else they are packed."""
    assert flmoe.fl_moe_debug_row_strides(cfg(hidden=hidden, dispatch_dtype=dtype)) == (dispatch, combine)


def test_row_strides_refuse_what_cannot_be():
    lib, v = flmoe.lib(), C.c_int64()
    assert lib.fl_moe_debug_row_strides(C.byref(cfg()), None, C.byref(v)) == flmoe.FL_ERR_INVALID_ARG
    assert lib.fl_moe_debug_row_strides(C.byref(cfg()), C.byref(v), None) == flmoe.FL_ERR_INVALID_ARG
    assert lib.fl_moe_debug_row_strides(C.byref(cfg(hidden=7)), C.byref(v), C.byref(v)) < 0


@pytest.mark.parametrize("N,El,T", [(64, 4, 4096), (32, 8, 8192), (32, 8, 2048), (1, 8, 1 << 20), (8, 16, 40000), (4, 4, 1),
                                    (64, 16, 3000)])
def test_every_counting_block_of_the_layout_owns_a_tile(N, El, T):
    for ranks in {1, N // 2 or 1, N}:
        plan = flmoe.fl_moe_debug_launch_plan(cfg(n_ranks=N, n_experts=N * El, max_tokens=T, hidden=8), ranks)
        blocks, tiles = plan.layout_blocks, plan.layout_tiles
        assert 1 <= blocks <= min(tiles, max(1, 512 // ranks - 1))          # with the planning blocks on 256 units
        per_block = -(-tiles // blocks)
        assert (blocks - 1) * per_block < tiles                             # the last block's first tile exists
        if tiles <= 512 // ranks - 1:
            assert blocks == tiles


def test_static_layout_entry_point_checks_its_arguments_before_touching_a_gpu():
    """fl_moe_layout_static validates on the host first: null or misaligned pointers, bad
    configurations and configurations beyond its static scratch array are refused without
    any device call (so this runs without a GPU)."""
    L = flmoe.lib()
    small = cfg(n_ranks=4, n_experts=32, max_tokens=64, top_k=4, hidden=256)
    fake = 0x1000                                   # never dereferenced: every call below fails earlier
    out = flmoe.fl_moe_layout_out(*([fake] * len(flmoe.LAYOUT_OUT_FIELDS)))
    assert L.fl_moe_layout_static(None, fake, fake, C.byref(out), None) == flmoe.FL_ERR_INVALID_ARG
    assert L.fl_moe_layout_static(C.byref(small), None, fake, C.byref(out), None) == flmoe.FL_ERR_INVALID_ARG
    assert L.fl_moe_layout_static(C.byref(small), fake, fake, None, None) == flmoe.FL_ERR_INVALID_ARG
    hole = flmoe.fl_moe_layout_out(*([fake] * (len(flmoe.LAYOUT_OUT_FIELDS) - 1) + [None]))
    assert L.fl_moe_layout_static(C.byref(small), fake, fake, C.byref(hole), None) == flmoe.FL_ERR_INVALID_ARG
    odd = flmoe.fl_moe_layout_out(*([fake + 2] + [fake] * (len(flmoe.LAYOUT_OUT_FIELDS) - 1)))
    assert L.fl_moe_layout_static(C.byref(small), fake, fake, C.byref(odd), None) == flmoe.FL_ERR_ALIGNMENT
    assert L.fl_moe_layout_static(C.byref(small), fake + 1, fake, C.byref(out), None) == flmoe.FL_ERR_ALIGNMENT
    bad = cfg(n_ranks=4, n_experts=30)
    assert L.fl_moe_layout_static(C.byref(bad), fake, fake, C.byref(out), None) == flmoe.FL_ERR_INVALID_ARG
    # the decode shape fits the array, the 4096-token shape does not (per-pair tables of 8 MB)
    big = cfg(max_tokens=4096)
    assert L.fl_moe_layout_static(C.byref(big), fake, fake, C.byref(out), None) == flmoe.FL_ERR_STATIC_LIMIT
    assert b"static" in L.fl_moe_strerror(flmoe.FL_ERR_STATIC_LIMIT)
    assert flmoe.FL_STATIC_SCRATCH_BYTES == 8 << 20


def test_host_only_queries_work_on_a_torch_without_gpu_functions():
    code = ("import torch\n"
            "for name in ('_cuda_getCurrentRawStream', '_cuda_getDevice'):\n"
            "    if hasattr(torch._C, name): delattr(torch._C, name)\n"
            "from paper_2510_27656_amd import flmoe\n"
            "c = flmoe.fl_moe_config(2, 8, 16, 2, 256, 0, 1, 0, 0, 0, 0, 0, 0)\n"
            "assert flmoe.fl_moe_query_sizes(c).workspace_bytes > 0\n")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT, timeout=100)


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    """(the compiler's resource report, the assembly) of the kernels in the tree."""
    from paper_2510_27656_amd import build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no compiler here")
    out = str(tmp_path_factory.mktemp("asm") / "kernels.s")
    report = subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                             "-packed-fp32-ops", "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-S", "-o",
                             out] + [os.path.join(build.CSRC, f) for f in build.SOURCES],
                            check=True, capture_output=True, text=True, timeout=300).stderr
    return report, open(out).read()


def test_no_kernel_spills_registers(compiled):
    """Scratch memory in a row loop costs more than any register saved."""
    names = re.findall(r"Function Name: (\S+)", compiled[0])
    scratch = [int(v) for v in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", compiled[0])]
    assert len(names) == len(scratch) >= 30
    assert not [n for n, v in zip(names, scratch) if v]


def test_two_workgroups_of_the_polling_reduce_kernel_fit_a_unit(compiled):
    """Its grid is capped, its workgroups have up to 16 waves: more than 64 registers halve the waves that sum."""
    registers = re.findall(r"Function Name: \S*combine_reduce_kernelILi1E.*?\bVGPRs: (\d+)", compiled[0], re.S)
    assert len(registers) == 6 and all(int(v) <= 64 for v in registers), registers


def test_nothing_overwrites_the_data_of_a_store_while_it_is_read(compiled):
    """Two wait states between a 128-bit store and a vector instruction that writes its data registers; the compiler
    keeps them only behind the stores that it makes itself."""
    code = [line.split(";")[0].strip() for line in compiled[1].splitlines()]
    code = [line for line in code if line and not line.startswith(".") or re.match(r"\.LBB\S*:$", line)]
    stores = [i for i, line in enumerate(code) if re.match(r"global_store_dwordx4 .*\bsc1\b", line)]
    assert len(stores) > 30
    for i in stores:
        first, last = map(int, re.search(r"\], v\[(\d+):(\d+)\]", code[i]).groups())
        states = 0
        for line in code[i + 1:]:
            nop = re.match(r"s_nop (\d+)", line)
            states += int(nop.group(1)) + 1 if nop else 0 if line.endswith(":") else 1
            if states >= 2:
                break
            for lo, hi in re.findall(r"^v_\S+ v\[?(\d+):?(\d*)", line):
                assert not (int(lo) <= last and int(hi or lo) >= first), (code[i], line)
            assert not line.startswith("s_cbranch") and not line.startswith("s_branch"), (code[i], line)


def test_loaded_library_was_built_from_the_sources_in_the_tree():
    from paper_2510_27656_amd import build
    assert flmoe.fl_moe_build_id() == build.source_hash() and len(build.source_hash()) == 16

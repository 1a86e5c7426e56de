"""The hand-placed LDS waits of the fused dK/dV kernel, checked on the compiler's listing (no GPU).

The kernel's operand reads are explicit instructions whose results the compiler does not track; the checker models
the LDS counter and flags any instruction that touches a register of a read still in flight.  The model itself is
pinned on small listings written here: a correct sequence, one with a wait count one too large, one where the
compiler would have moved a copy in front of the wait.
"""
import functools
import os
import re

import pytest

from paper_2409_15373_amd import build, check_lds_waits

GOOD = """
    ds_read_b128 v[4:7], v1
    ds_read_b128 v[8:11], v1 offset:32
    ds_read_b128 v[12:15], v1 offset:64
    s_waitcnt lgkmcnt(2)
    v_mfma_f32_32x32x16_bf16 v[20:35], v[4:7], v[40:43], v[20:35]
    s_waitcnt lgkmcnt(1)
    v_mfma_f32_32x32x16_bf16 v[20:35], v[8:11], v[44:47], v[20:35]
    s_waitcnt lgkmcnt(0)
    v_mfma_f32_32x32x16_bf16 v[20:35], v[12:15], v[48:51], v[20:35]
"""


def test_a_correct_sequence_passes():
    r = check_lds_waits.scan(GOOD)
    assert r["violations"] == [] and r["lds_reads"] == 3 and r["lgkmcnt_waits"] == 3 and r["deepest_queue"] == 3


def test_a_count_one_too_large_is_found():
    r = check_lds_waits.scan(GOOD.replace("s_waitcnt lgkmcnt(1)", "s_waitcnt lgkmcnt(2)"))
    assert len(r["violations"]) == 1 and "v[8:11]" in r["violations"][0][1]


def test_a_copy_of_a_pending_register_is_found():
    r = check_lds_waits.scan(GOOD.replace("    s_waitcnt lgkmcnt(2)\n", "    v_mov_b32_e32 v60, v13\n    s_waitcnt lgkmcnt(2)\n"))
    assert len(r["violations"]) == 1 and "v_mov_b32" in r["violations"][0][1]


def test_a_store_in_the_queue_counts():
    # operations complete in order: with a write issued after the read, lgkmcnt(1) is enough for the read; without it, it is not
    with_store = "    ds_read_b128 v[4:7], v1\n    ds_write_b32 v2, v3\n    s_waitcnt lgkmcnt(1)\n    v_mov_b32_e32 v9, v4\n"
    assert check_lds_waits.scan(with_store)["violations"] == []
    assert len(check_lds_waits.scan(with_store.replace("    ds_write_b32 v2, v3\n", ""))["violations"]) == 1


def test_scalar_loads_are_ignored_and_overwrites_are_found():
    r = check_lds_waits.scan("    ds_read_b64_tr_b16 v[4:5], v1\n    s_load_dword s4, s[0:1], 0x0\n    v_mov_b32_e32 v5, 0\n    s_waitcnt lgkmcnt(0)\n")
    assert len(r["violations"]) == 1


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_the_fused_kernel_reads_no_register_in_flight():
    r = check_lds_waits.scan(check_lds_waits.listing_of(os.path.join(build.CSRC, "jfa_bwd_dkv_dma.hip")))
    assert r["lds_reads"] > 1000 and r["violations"] == [], r["violations"][:5]
    assert r["deepest_queue"] <= 15   # the counter has four bits


def test_partial_vmcnt_model_counts_what_follows_a_wait():
    text = """
        s_waitcnt vmcnt(2) lgkmcnt(0)
        global_load_lds_dwordx4 v1, s[2:3]
        global_store_dwordx4 v[2:3], v[4:7], off
        scratch_load_dword v9, off, off
        global_store_dwordx4 v[2:3], v[4:7], off
        s_barrier
        global_store_dwordx4 v[2:3], v[4:7], off
    """
    assert check_lds_waits.behind_partial_vmcnt_wait(text, 2) == [(1, 2, 1)]
    assert check_lds_waits.behind_partial_vmcnt_wait(text, 3) == []


def test_the_few_query_backward_leaves_exactly_its_stores_in_flight():
    """Its wait for a block's K and V rows is vmcnt(16): sixteen copies of the next block, then the sixteen stores of
    dK and dV that may stay in flight, and no other vector-memory instruction (no scratch) in the block loop."""
    listing = check_lds_waits.listing_of(os.path.join(build.CSRC, "jfa_bwd_cross_fewq.hip"))
    assert check_lds_waits.behind_partial_vmcnt_wait(listing, 16) == [(16, 16, 0)]


def test_scalar_operand_model():
    close = """
        v_readlane_b32 s5, v255, 18
        s_mov_b32 m0, s1
        s_nop 0
        global_load_lds_dword v0, s[4:5]
    """
    assert [h[2] for h in check_lds_waits.scalar_operand_hazards(close)] == [2]
    assert check_lds_waits.scalar_operand_hazards(close.replace("s_nop 0", "s_nop 3")) == []
    assert len(check_lds_waits.scalar_operand_hazards(close.replace("s_nop 0", "s_nop 2"))) == 1
    # a scalar instruction that writes the register in between: the vector instruction's value is not what is read
    assert check_lds_waits.scalar_operand_hazards(close.replace("s_nop 0", "s_mov_b64 s[4:5], s[8:9]")) == []
    # another register, or a vector address
    assert check_lds_waits.scalar_operand_hazards(close.replace("s[4:5]", "s[6:7]")) == []


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("source", check_lds_waits.HAND_WRITTEN_COPIES)
def test_no_copy_reads_its_scalar_base_too_early(source):
    """The base of a hand-written copy may come out of a spill (v_readlane) right in front of it; the copy itself has to bring
    the wait states that the hardware needs between the two."""
    listing = check_lds_waits.listing_of(os.path.join(build.CSRC, source))
    assert "global_load_lds" in listing
    assert check_lds_waits.scalar_operand_hazards(listing) == []


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_the_head_size_64_gradient_kernels_use_no_scratch_memory():
    """Spilled registers cost every launch of these kernels 4 us, a fifth of a small batch's dQ."""
    listing = check_lds_waits.listing_of(os.path.join(build.CSRC, "jfa_bwd_narrow.hip"))
    sizes = dict(re.findall(r"\.amdhsa_kernel (\S*Li64\S*)\s+(?:\.\S.*\s+)*?\.amdhsa_private_segment_fixed_size (\d+)", listing))
    assert len(sizes) == 6 and set(sizes.values()) == {"0"}, sizes


listing_of = functools.lru_cache(maxsize=None)(check_lds_waits.listing_of)


def scratch_sizes(source, kernel):
    """{template arguments as mangled: bytes of scratch per lane} of a kernel's instances"""
    listing = listing_of(os.path.join(build.CSRC, source))
    found = re.findall(r"\.amdhsa_kernel \S*%sI(\S*?)EEv\S*\s+(?:\.\S.*\s+)*?\.amdhsa_private_segment_fixed_size (\d+)" % kernel, listing)
    return {args: int(size) for args, size in found}


NARROW_BACKWARD = ["jfa_bwd_narrow.hip", "jfa_bwd_narrow_direct.hip"]


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("sources,kernel,direct,scheduled", [
    (["jfa_fwd_bf16_dma.hip"], "fwd_bf16_dma_kernel", "Lb1", "Lb0"), (["jfa_bwd_dq_dma.hip"], "bwd_dq_dma_kernel", "Lb1", "Lb0"),
    (["jfa_bwd_dkv_dma.hip"], "bwd_dkv_dma_kernel", "Li1", "Li0|Lin1"), (["jfa_fwd_narrow.hip"], "fwd_narrow_kernel", "Li1", "Li0"),
    (NARROW_BACKWARD, "dq_narrow_kernel", "Li1", "Li0|Lin1"), (NARROW_BACKWARD, "dkv_narrow_kernel", "Li1", "Li0|Lin1")])
def test_calls_without_a_schedule_have_instances_of_their_own(sources, kernel, direct, scheduled):
    """The walk without a schedule beside the one with it costs both of them registers: apart, the former uses no more scratch memory."""
    sizes = {}
    for source in sources:
        sizes.update(scratch_sizes(source, kernel))
    pairs = 0
    for args, size in sizes.items():
        form = re.fullmatch(r"(.*E)(%s)E" % direct, args)
        if form:
            pairs += 1
            assert size <= min(s for a, s in sizes.items() if re.fullmatch(re.escape(form.group(1)) + "(%s)E" % scheduled, a)), sizes
    assert pairs >= 2, sizes


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("source", NARROW_BACKWARD)
@pytest.mark.parametrize("kernel", ["dq_narrow_kernel", "dkv_narrow_kernel"])
def test_the_head_size_32_gradient_kernels_use_no_scratch_memory(source, kernel):
    sizes = {a: n for a, n in scratch_sizes(source, kernel).items() if a.startswith("Li32")}
    assert len(sizes) == 3 and set(sizes.values()) == {0}, sizes

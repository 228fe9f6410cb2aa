"""Promises of the matrix products that the compiler does not check, in the code built for the GPU."""
import re

import gpu_code


def test_alternating_tiles_keep_their_registers(tmp_path):
    """Two k-tiles a round of the main loop are for the tiles whose registers hold the second set of addresses.  (256x256 tiles on the 16x16x32 instruction with the epilogue of kind 4
    keep two of a lane's values in scratch with either loop.)"""
    seen, spilled = 0, []
    for co in gpu_code.code_objects(tmp_path):
        for name, r in gpu_code.resources(co).items():
            if "gemm_pp" not in name:
                continue
            seen += 1
            if r["private_segment_fixed_size"] > (8 if "PpTileILi256ELi128ELi128ELi4ELi2ELi16EEELi4ELb0ELb0ELb0E" in name else 0):
                spilled.append((name, r))
    assert seen > 100 and not spilled, spilled


def _states(code):
    """Wait states that an instruction makes for the ones behind it."""
    nop = re.fullmatch(r"s_nop (\d+)", code)
    return int(nop.group(1)) + 1 if nop else 1


def test_closing_a_segment_waits_for_the_products(tmp_path):
    """The sums of a segment are added to the total and cleared by instructions that the compiler counts no wait states for.  Straight in front of the first of them are the 19
    that the longest matrix instruction asks for before its result is read, straight behind the last the 8 for the next one to take the zeros, and no matrix instruction is
    in between."""
    closings = 0
    for co in gpu_code.code_objects(tmp_path):
        for name, body in gpu_code.listings(co, lambda n: "gemm_bf16_dtl_kernel" in n):
            pairs = []
            for i in range(len(body) - 1):
                add = re.fullmatch(r"v_add_f32(?:_e32)? (v\d+), \1, (v\d+)", body[i])
                if add and re.fullmatch(rf"v_mov_b32(?:_e32)? {add.group(2)}, 0", body[i + 1]):
                    pairs.append(i)
            at = 0
            while at < len(pairs):
                first = last = at
                while last + 1 < len(pairs) and not any(_states(c) >= 8 for c in body[pairs[last]:pairs[last + 1]]):
                    last += 1
                before = after = 0
                k = pairs[first] - 1
                while k >= 0 and body[k].startswith("s_nop"):
                    before += _states(body[k])
                    k -= 1
                for code in body[pairs[last] + 2:]:
                    if not code.startswith("s_nop"):
                        break
                    after += _states(code)
                inside = body[pairs[first]:pairs[last]]
                assert before >= 19 and after >= 8 and (last - first + 1) % 16 == 0, (name, before, after, last - first + 1)
                assert not any(c.startswith(("v_mfma", "v_smfma", "s_cbranch", "s_branch")) for c in inside), name
                closings += 1
                at = last + 1
    assert closings >= 45, closings      # two or three in each of fifteen kernels and more

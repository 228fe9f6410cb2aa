"""Promises of the matrix products that the compiler does not check, in the code built for the GPU."""
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

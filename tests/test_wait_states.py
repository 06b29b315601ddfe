"""The built kernels keep the wait states that the hardware does not, on every path: walks over the disassembly of libaquakv.so.

* Between a matrix instruction and the vector instructions that read its result, from each v_mfma_f32_32x32x16_bf16 (8 passes: 12 states,
  which is what the compiler keeps on the paths that it counts).
* Between a vector instruction and the lane permutes (DPP) and lane swaps (v_permlane*) that read its result: 2 states.  The compiler
  keeps them between instructions of its own and does not look into assembly, so blocks of assembly carry them at their edges.
* LDS words that assembly requests and waits for later are left alone until they have arrived.

One walk looks at an order that speed depends on and that the compiler is free to turn round."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2501_19392_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
STATES = 12
OPERAND = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))")
STORES = ("global_store", "ds_write", "buffer_store", "scratch_store", "flat_store")


def registers(text):
    out = set()
    for kind, first, last, one in OPERAND.findall(text):
        out.update((kind, i) for i in range(int(first or one), int(last or one) + 1))
    return out


def functions(listing):
    """(name, [(mnemonic, operands)], {label: index}) per function"""
    name, code, labels = None, [], {}
    for line in listing:
        if m := re.match(r"[0-9a-f]+ <(_Z\w+)>:", line):
            if name:
                yield name, code, labels
            name, code, labels = m[1], [], {}
        elif m := re.match(r"(?:[0-9a-f]+ )?<(L\d+)>:", line):
            labels[m[1]] = len(code)
        elif m := re.match(r"\s+([a-z]\w+)\s*(.*?)\s*(?://.*)?$", line):
            code.append((m[1], m[2]))
    if name:
        yield name, code, labels


def shortest(code, labels, start):
    """Wait states from the matrix instruction at `start` to the first read of its result, at most STATES are looked at."""
    result = registers(code[start][1].split(",")[0])
    best, seen, paths = STATES, {}, [(start + 1, 0)]
    while paths:
        at, w = paths.pop()
        while at < len(code) and w < best and seen.get(at, STATES) > w:
            seen[at] = w
            op, args = code[at]
            if op.startswith("v_mfma") or op == "s_endpgm":          # (matrix instructions wait for one another in hardware)
                if op == "s_endpgm":
                    break
            elif registers(args if op.startswith(STORES) else args.partition(",")[2]) & result:
                best = w
                break
            w += int(args, 0) + 1 if op == "s_nop" else 1
            target = labels[re.search(r"L\d+", args)[0]] if op == "s_branch" or op.startswith("s_cbranch") else None
            if op == "s_branch":
                at = target
                continue
            if target is not None:
                paths.append((target, w))
            at += 1
    return best


def permutes(op, args):
    return op.startswith("v_permlane") or op.endswith("_dpp") or "quad_perm" in args or " row_" in args


def results(op, args):
    """Vector registers that a vector instruction writes; a lane swap writes both of its operands."""
    if not op.startswith("v_") or op.startswith("v_mfma"):
        return set()
    return registers(",".join(args.split(",")[:2 if op.startswith("v_permlane") or op == "v_swap_b32" else 1]))


def permuted_early(code, labels, start, states=2):
    """Whether a lane permute or swap reads a result of the vector instruction at `start` before `states` have passed."""
    result, paths = results(*code[start]), [(start + 1, 0)]
    while paths:
        at, w = paths.pop()
        while at < len(code) and w < states and code[at][0] != "s_endpgm":
            op, args = code[at]
            if permutes(op, args) and registers(args) & result:
                return True
            w += int(args, 0) + 1 if op == "s_nop" else 1
            if op == "s_branch" or op.startswith("s_cbranch"):
                paths.append((labels[re.search(r"L\d+", args)[0]], w))
                if op == "s_branch":
                    break
            at += 1
    return False


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    """functions() of every code object in the library"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    tmp_path = tmp_path_factory.mktemp("objects")
    shutil.copy(B.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    out = []
    for obj in sorted(tmp_path.glob("lib.so.*gfx950")):
        out += functions(subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", str(obj)], check=True, capture_output=True,
                                        text=True).stdout.splitlines())
    return out


def test_results_of_matrix_instructions_are_not_read_early(built):
    checked = 0
    for name, code, labels in built:
        for i, (op, _) in enumerate(code):
            if op == "v_mfma_f32_32x32x16_bf16":
                checked += 1
                assert shortest(code, labels, i) >= STATES, (name, i)
    assert checked > 1000


def test_results_of_vector_instructions_are_not_permuted_early(built):
    swaps = 0
    for name, code, labels in built:
        near = [False] * (len(code) + 2)                 # a permute, or a branch that may lead to one, is among the next two
        for i, (op, args) in enumerate(code):
            swaps += op.startswith("v_permlane")
            if permutes(op, args) or op.startswith(("s_branch", "s_cbranch")):
                near[max(i - 1, 0)] = near[max(i - 2, 0)] = True
        for i, (op, args) in enumerate(code):
            if near[i] and results(op, args):
                assert not permuted_early(code, labels, i), (name, i, code[i:i + 4])
    assert swaps > 1000


def test_assembly_ahead_of_lane_swaps_ends_with_wait_states(built):
    """The stage of the transform that lane swaps follow: 16 multiply-adds in one block, whichever instruction comes after it."""
    blocks = 0
    for name, code, _ in built:
        run = 0
        for i, (op, args) in enumerate(code):
            if op == "v_fmac_f32_dpp" and "row_ror:8" in args:
                run += 1
                if run % 16 == 0:
                    blocks += 1
                    assert code[i + 1][0] == "s_nop" and int(code[i + 1][1], 0) >= 1, (name, i, code[i:i + 3])
    assert blocks > 10


def test_lds_words_requested_by_assembly_are_left_alone(built):
    """The main loop of the stand-alone predictor posts its count (ds_write_b32) and requests the team's four (ds_read_b128), which
    arrive by the next wait for all of the LDS: nothing else reads or writes their registers before, whichever way the code goes."""
    requests = 0
    for name, code, labels in built:
        if "predict_bf16_kernel" not in name:
            continue
        for i, (op, args) in enumerate(code):
            if op != "ds_read_b128" or "offset" in args or not any(o == "ds_write_b32" for o, _ in code[max(i - 6, 0):i]):
                continue
            requests += 1
            words, seen, paths = registers(args.split(",")[0]), set(), [i + 1]
            while paths:
                at = paths.pop()
                while at not in seen:
                    seen.add(at)
                    op, args = code[at]
                    if op == "s_waitcnt" and "lgkmcnt(0)" in args:
                        break
                    assert op != "s_endpgm" and not registers(args) & words, (name, i, at, code[at])
                    if op == "s_branch" or op.startswith("s_cbranch"):
                        paths.append(labels[re.search(r"L\d+", args)[0]])
                        if op == "s_branch":
                            break
                    at += 1
    assert requests >= 2


def test_uniform_quantizers_stage_no_search_table(built):
    """A round-to-nearest layer's grid pointers may hold anything: its encoders do not fetch a search table, whose way to LDS is the only
    use of 16-byte stores there (a grid's encoders have them)."""
    stores = {}
    for name, code, _ in built:
        if m := re.search(r"(fused_kernel|fused_two_heads_kernel|fused_tile_kernel|fused_tile_two_kernel|fused_tile_pair_kernel)ILi(\d+)ELi0E", name):
            stores.setdefault((m[1], int(m[2]) in (2, 4)), []).append(sum(op == "ds_write_b128" for op, _ in code))
    assert len(stores) == 10
    for (kernel, uniform), counts in stores.items():
        assert not any(counts) if uniform else all(counts), (kernel, uniform, counts)


def test_rows_written_past_the_caches(built):
    """Tiles of 256 rows and whole tokens write large launches past the L2s and others through them (a branch of the kernel); the readers of the
    other tiles' rows are slower for it at every size, so those have no such store."""
    past = {}
    for name, code, _ in built:
        if m := re.search(r"(fused_kernel|fused_two_heads_kernel|fused_wide_encode_kernel|fused_tile_kernel|fused_tile_two_kernel|fused_tile_pair_kernel|"
                          r"fused_tile_attend_kernel|quantize_kernel)I", name):
            stores = [args for op, args in code if op == "global_store_dwordx4"]
            past.setdefault(m[1], []).append((sum(args.endswith(" nt") for args in stores), len(stores)))
    assert len(past) == 8
    for kernel, counts in past.items():
        asks = kernel in ("fused_kernel", "fused_two_heads_kernel", "fused_wide_encode_kernel")
        assert all(0 < nt < all_stores if asks else nt == 0 for nt, all_stores in counts), (kernel, counts)


def test_waves_that_multiply_issue_no_loads(built):
    """In the steady loop of a tile's multiplying waves every load is another wave's: four matrix instructions (k 64) for each block of the
    wave, its fragments from LDS, one barrier, and at most one address addition for each k step and operand."""
    checked = 0
    for name, code, labels in built:
        if not (m := re.search(r"fused_tile(_pair)?_kernelILi\d+ELi\dELi(\d+)E", name)):
            continue
        starts = sorted({0, *labels.values(), len(code)})
        for begin, end in zip(starts, starts[1:]):
            ops = [op for op, _ in code[begin:end]]
            if ops.count("s_barrier") == 1 and ops.count("v_mfma_f32_32x32x16_bf16") == 4 * int(m[2]):
                checked += 1
                assert not any(op.startswith(("global_load", "buffer_load")) for op in ops), (name, begin)
                assert ops.count("v_add_u32_e32") <= 8, (name, begin)
    assert checked > 150


# kernels built on the loop with loading waves, and the row blocks of their tiles
TILE_KERNELS = [(r"fused_tile_kernelILi\d+ELi\dELi(\d+)E", None), (r"fused_tile_two_kernelILi\d+ELi\dELi(\d+)E", None),
                (r"predict_two_tiles_kernelILi(\d+)ELi(\d+)E", None), (r"fused_tile_pair_kernelILi", 1), (r"fused_kernelILi", 8), (r"fused_attend_kernelILi", 8),
                (r"fused_tile_attend_kernelILi\d+ELi(\d+)E", None)]


def test_steady_loops_of_every_kernel_on_tiles(built):
    """Every kernel on tiles: in each steady loop of its multiplying waves no load, a k-tile's fragments from LDS (four steps of the wave's blocks
    of rows and of columns) and nothing more, one barrier."""
    found = {}
    for name, code, labels in built:
        for pattern, fixed in TILE_KERNELS:
            if not (m := re.search(pattern, name)):
                continue
            for blocks in (map(int, m.groups()) if fixed is None else [fixed]):
                reads = 4 * (blocks + 1 if blocks < 4 else blocks // 2 + 2)
                loops = 0
                starts = sorted({0, *labels.values(), len(code)})
                for begin, end in zip(starts, starts[1:]):
                    ops = [op for op, _ in code[begin:end]]
                    if ops.count("s_barrier") == 1 and ops.count("v_mfma_f32_32x32x16_bf16") == 4 * blocks:
                        loops += 1
                        assert not any(op.startswith(("global_load", "buffer_load")) for op in ops), (name, begin)
                        assert ops.count("ds_read_b128") == reads and not any(op.startswith("ds_write") for op in ops), (name, begin, ops.count("ds_read_b128"))
                assert loops >= 1, (name, blocks)
                found[pattern] = found.get(pattern, 0) + 1
    assert len(found) == len(TILE_KERNELS), found

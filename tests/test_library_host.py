"""CPU-side tests of the C-ABI library: it loads, exports every symbol the header
declares, sizes its workspace, and rejects bad arguments before touching a GPU."""
import ctypes
import os
import re
import shutil
import struct
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2605_18753_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def params(**kw):
    p = B.dash_params()
    base = dict(batch=1, h_q=8, h_kv=2, n_q=1024, n_kv=1024, head_dim=128, block_size=64, causal=1,
                dtype=B.DASH_BF16, alpha=1.5, gamma=1.0, sigma=1.0, scale=0.0)
    base.update(kw)
    for k, v in base.items():
        setattr(p, k, v)
    for name, heads, n in (("q_stride", p.h_q, p.n_q), ("k_stride", p.h_kv, p.n_kv),
                           ("v_stride", p.h_kv, p.n_kv), ("o_stride", p.h_q, p.n_q)):
        getattr(p, name)[:] = [heads * n * p.head_dim, n * p.head_dim, p.head_dim]
    return p


def header_functions():
    text = open(os.path.join(ROOT, "include", "dash_attn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return set(re.findall(r"\b(dash_\w+|dense_attn)\s*\(", text))


def test_library_exports_every_declared_symbol():
    lib = B.load_library()
    names = header_functions()
    assert {"dash_attn_prefill", "dash_attn_decode", "dense_attn", "dash_kbar_compress",
            "dash_kbar_summarize"} <= names
    for n in names:
        assert hasattr(lib, n), n
    assert names == set(B.exported_symbols())


def test_workspace_and_list_sizes():
    p = params()
    assert B.list_stride(p) == 16 and B.mask_words(p) == 1
    n = B.workspace_bytes(p)
    rows = 2 * 1024
    assert n >= rows * 16 * 4 + rows * 4 + 2 * 16 * 3 * 128 * 2
    p2 = params(n_q=1000, n_kv=1000)          # ragged tail: 15 complete chunks + 1 partial
    assert B.list_stride(p2) == 16
    pd = params(n_q=1, n_kv=131072, batch=16, h_q=32, h_kv=8)
    assert B.list_stride(pd) == 2048 and B.mask_words(pd) == 64
    # a decode step keeps its scores on chip: the bias lists and the split-KV partials are what it needs
    assert 16 * 8 * 2048 * 4 < B.workspace_bytes(pd) < 16 * 32 * 2047 * 4


def test_prefill_workspace_follows_the_shape():
    """A prefill needs room for the records of cut chunk lists only as far as it, or a smaller call in the same
    workspace, can be cut: nothing below 16 tiles of 64 keys, at most 1536 records of 128 rows."""
    size = lambda n, **kw: B.workspace_bytes(params(**{**dict(h_q=32, h_kv=8, n_q=n, n_kv=n), **kw}))
    lists = lambda n, h_kv=8: h_kv * (n // 64) * 3 * 128 * 2 + h_kv * n * ((n + 63) // 64 + (n + 2047) // 2048) * 4 + 4 * 256
    record = 128 * 130 * 4
    for n in (2, 100, 700, 960):
        assert size(n) <= lists(n), n
    assert size(1000) <= lists(1000) + 4096 + 256 * record
    assert size(2000) <= lists(2000) + 4096 + 512 * record
    assert size(1024, h_q=1, h_kv=1) <= lists(1024, 1) + 4096 + 16 * record        # 8 row tiles in two parts
    assert size(32768) <= lists(32768) + 4096 + 1536 * record
    # a workspace made for a larger call serves the smaller ones
    for h_q, h_kv in ((32, 8), (2, 2), (16, 1), (128, 64)):
        for d in (64, 128):
            for blk in (64, 128):
                get = lambda b, n_q, n_kv: B.workspace_bytes(params(batch=b, h_q=h_q, h_kv=h_kv, n_q=n_q, n_kv=n_kv, head_dim=d, block_size=blk))
                last = 0
                for n in list(range(64, 4096, 64)) + [8192, 30000, 131072]:
                    now = get(1, n, n)
                    assert now >= last, (h_q, h_kv, d, blk, n)
                    last = now
                    for n_q in (2, 64, 65, 600, 2000, 4096):
                        if n_q < n and (n - n_q) % 64 == 0:
                            assert get(1, n_q, n) <= now and now <= get(2, n, n)


@pytest.mark.parametrize("kw,code", [
    (dict(h_q=7), -1), (dict(alpha=1.0), -1), (dict(alpha=0.5), -1), (dict(sigma=0.0), -1),
    (dict(gamma=-1.0), -1), (dict(batch=0), -1), (dict(n_q=2048), -1), (dict(causal=2), -1),
    (dict(dtype=3), -1), (dict(causal=0, n_q=1000, n_kv=1000), -1),
    (dict(window=-1), -1), (dict(window=9), -1), (dict(window=1, causal=0), -1),
    (dict(head_dim=96), -2), (dict(block_size=32), -2), (dict(h_q=64, h_kv=2), -2),
    (dict(n_q=100, n_kv=1001), -2), (dict(n_q=262144, n_kv=262144), -2),
])
def test_invalid_parameters_are_rejected(kw, code):
    lib = B.load_library()
    p = params(**kw)
    # every compute entry point rejects the same way, before any launch
    assert lib.dash_attn_prefill(ctypes.byref(p), 256, 256, 256, 256, 256, None, None, None, None, None,
                                 256, 1 << 40, None) == code
    assert lib.dash_stage1_route(ctypes.byref(p), 256, 256, None, None, None, None, None,
                                 256, 1 << 40, None) == code
    if not (kw.get("causal") == 0 and len(kw) == 3):     # ragged non-causal is fine for dense
        n = ctypes.c_size_t(0)
        assert lib.dash_attn_workspace_bytes(ctypes.byref(p), ctypes.byref(n)) == code
        assert lib.dense_attn(ctypes.byref(p), 1, 1, 1, 1, 256, 1 << 40, None) == code


def test_null_and_workspace_errors():
    lib = B.load_library()
    p = params()
    need = B.workspace_bytes(p)
    assert lib.dense_attn(ctypes.byref(p), None, 1, 1, 1, 256, need, None) == -1
    assert lib.dense_attn(ctypes.byref(p), 256, 256, 256, 256, None, need, None) == -3
    assert lib.dense_attn(ctypes.byref(p), 256, 256, 256, 256, 256, need - 1, None) == -3
    assert lib.dense_attn(ctypes.byref(p), 256, 256, 256, 256, 257, need, None) == -3     # misaligned
    assert lib.dash_attn_prefill(ctypes.byref(p), 256, 256, 256, 256, None, None, None, None, None, None,
                                 256, need, None) == -1                                  # kbar is required
    assert lib.dash_attn_decode(ctypes.byref(p), 256, 256, 256, 256, 256, None, None, None, None, None,
                                256, need, None) == -1                                   # n_q must be 1
    assert lib.dash_attn_workspace_bytes(None, None) == -1
    p.q_stride[2] = 100                                                                    # misaligned rows
    assert lib.dense_attn(ctypes.byref(p), 256, 256, 256, 256, 256, need, None) == -1


def test_summarize_argument_errors():
    lib = B.load_library()
    p = params()
    ok = (ctypes.c_int64 * 3)(0, 128, 0)
    assert lib.dash_kbar_summarize(ctypes.byref(p), 256, None, ok, 256, 0, -1, None) == -1     # no query
    assert lib.dash_kbar_summarize(ctypes.byref(p), 256, 256, None, 256, 0, -1, None) == -1    # no strides
    assert lib.dash_kbar_summarize(ctypes.byref(p), 256, 264, ok, 256, 0, -1, None) == -1      # query not 16-byte aligned
    assert lib.dash_kbar_summarize(ctypes.byref(p), 256, 256, (ctypes.c_int64 * 3)(0, 100, 0), 256, 0, -1,
                                   None) == -1                                                # stride not a multiple of 8
    assert lib.dash_kbar_summarize(ctypes.byref(p), 256, 256, (ctypes.c_int64 * 3)(0, -128, 0), 256, 0, -1,
                                   None) == -1
    assert lib.dash_kbar_summarize(ctypes.byref(p), 256, 256, ok, 256, 15, 2, None) == -1      # 16 chunks: 15..16
    assert lib.dash_kbar_summarize(ctypes.byref(p), 256, 256, ok, 256, 3, 0, None) == 0        # empty range: nothing to do
    assert lib.dash_kbar_compress(ctypes.byref(p), 256, 256, 15, 2, None) == -1


def test_ragged_decode_argument_errors():
    lib = B.load_library()
    p = params(n_q=1, n_kv=4096)
    need = B.workspace_bytes(p)
    args = (256, 256, 256, 256)
    assert lib.dash_attn_decode_ragged(ctypes.byref(p), *args, None, 1, 256, None, None, None, None, None,
                                       256, need, None) == -1                            # no lengths
    p32 = params(n_q=1, n_kv=4096, dtype=0)
    assert lib.dash_attn_decode_ragged(ctypes.byref(p32), *args, 256, 1, 256, None, None, None, None, None,
                                       256, 1 << 40, None) == -2                          # bf16 only
    pq = params(n_q=64, n_kv=4096)
    assert lib.dash_attn_decode_ragged(ctypes.byref(pq), *args, 256, 1, 256, None, None, None, None, None,
                                       256, 1 << 40, None) == -1                          # one query per sequence


def test_backward_argument_errors():
    lib = B.load_library()
    p = params()
    need = B.backward_workspace_bytes(p)
    assert need > 2 * 8 * 1024 * 4 + 8 * 1024 * 128 * 4
    ptrs = [256] * 12          # q k v d_o kbar mask bias tau dq dk dv dkbar
    for i in range(11):          # the last one (dkbar) is optional
        bad = list(ptrs)
        bad[i] = None
        assert lib.dash_attn_backward(ctypes.byref(p), *bad, 256, need, None) == -1, i
    assert lib.dash_attn_backward(ctypes.byref(p), *ptrs, None, need, None) == -3
    assert lib.dash_attn_backward(ctypes.byref(p), *ptrs, 256, need - 1, None) == -3
    assert lib.dash_attn_backward(ctypes.byref(p), *ptrs, 257, need, None) == -3
    n = ctypes.c_size_t(0)
    pu = params(n_q=512, n_kv=1024)                                 # a chunked prefill
    assert lib.dash_attn_backward_workspace_bytes(ctypes.byref(pu), ctypes.byref(n)) == -2
    assert lib.dash_attn_backward(ctypes.byref(pu), *ptrs, 256, 1 << 40, None) == -2
    assert lib.dash_attn_backward_workspace_bytes(ctypes.byref(params(dtype=0)), ctypes.byref(n)) == 0   # fp32 tensors
    assert n.value == need
    assert lib.dash_attn_backward_workspace_bytes(ctypes.byref(p), None) == -1
    big = params(h_q=16, h_kv=1, n_q=131072, n_kv=131072)          # a 16-head slice of q spans 512 MiB: fine
    assert lib.dash_attn_backward_workspace_bytes(ctypes.byref(big), ctypes.byref(n)) == 0
    far = params()
    far.q_stride[1] = 1 << 31                                       # heads 4 GiB apart: 32-bit offsets do not reach
    assert lib.dash_attn_backward_workspace_bytes(ctypes.byref(far), ctypes.byref(n)) == -2


def test_forward_rejects_slices_beyond_32_bit_offsets():
    """The bf16 kernels address one (batch, kv-head) slice of a tensor with 32-bit byte offsets:
    a token-major cache whose slice spans 2 GiB or more is refused by every forward entry point
    (fp32 tensors use 64-bit offsets and are accepted)."""
    lib = B.load_library()
    n = ctypes.c_size_t(0)
    ok = params(n_q=1, n_kv=131072, batch=16, h_q=32, h_kv=8)
    ok.k_stride[2] = ok.v_stride[2] = 8 * 128                     # [batch, token, head, d]: 268 MB per slice
    ok.k_stride[1] = ok.v_stride[1] = 128
    assert lib.dash_attn_workspace_bytes(ctypes.byref(ok), ctypes.byref(n)) == 0
    for name in ("k_stride", "v_stride", "q_stride", "o_stride"):
        wide = params(n_q=8192, n_kv=8192)
        getattr(wide, name)[2] = 1 << 18                           # 8191 * 512 KiB + 256 B >= 2 GiB
        assert lib.dash_attn_workspace_bytes(ctypes.byref(wide), ctypes.byref(n)) == -2, name
        assert lib.dash_attn_prefill(ctypes.byref(wide), 256, 256, 256, 256, 256, None, None, None, None, None,
                                     256, 1 << 40, None) == -2, name
        assert lib.dense_attn(ctypes.byref(wide), 256, 256, 256, 256, 256, 1 << 40, None) == -2, name
        assert lib.dash_stage2_attend(ctypes.byref(wide), 256, 256, 256, 256, None, None, 256, 1 << 40, None) == -2
        wide.dtype = 0                                             # fp32: plain 64-bit pointers
        getattr(wide, name)[2] = 1 << 18
        assert lib.dash_attn_workspace_bytes(ctypes.byref(wide), ctypes.byref(n)) == 0, name
    dec = params(n_q=1, n_kv=131072, batch=2, h_q=8, h_kv=2)
    dec.k_stride[2] = 1 << 14                                      # 131071 * 32 KiB >= 2 GiB
    assert lib.dash_attn_decode(ctypes.byref(dec), 256, 256, 256, 256, 256, None, None, None, None, None,
                                256, 1 << 40, None) == -2
    heads = params()
    heads.q_stride[1] = 1 << 30                                    # the 4 query heads of a kv-head 2 GiB apart
    assert lib.dash_attn_workspace_bytes(ctypes.byref(heads), ctypes.byref(n)) == -2


def test_backward_is_refused_above_the_alpha_it_is_checked_to():
    lib = B.load_library()
    n = ctypes.c_size_t(0)
    assert lib.dash_attn_backward_workspace_bytes(ctypes.byref(params(alpha=3.0)), ctypes.byref(n)) == 0
    assert lib.dash_attn_backward_workspace_bytes(ctypes.byref(params(alpha=4.0)), ctypes.byref(n)) == -2
    assert lib.dash_attn_backward(ctypes.byref(params(alpha=4.0)), *([256] * 12), 256, 1 << 40, None) == -2
    # the forward has no such limit
    assert lib.dash_attn_workspace_bytes(ctypes.byref(params(alpha=4.0)), ctypes.byref(n)) == 0


def test_the_library_reads_no_environment_variable():
    """Behaviour depends on the arguments alone: the sources call no getenv."""
    csrc = os.path.join(ROOT, "paper_2605_18753_amd", "csrc")
    for f in os.listdir(csrc):
        if f.endswith((".hip", ".h")):
            assert "getenv" not in open(os.path.join(csrc, f)).read(), f


def test_summarize_backward_argument_errors():
    lib = B.load_library()
    p = params()
    ok = (ctypes.c_int64 * 3)(0, 128, 0)
    good = [256, 256, ok, 256, 256, 256]         # k qbar strides dkbar dk dqbar
    for i in range(6):
        bad = list(good)
        bad[i] = None
        assert lib.dash_kbar_summarize_backward(ctypes.byref(p), *bad, None) == -1, i
    assert lib.dash_kbar_summarize_backward(ctypes.byref(p), 256, 264, ok, 256, 256, 256, None) == -1   # alignment
    assert lib.dash_kbar_summarize_backward(ctypes.byref(p), 256, 256, (ctypes.c_int64 * 3)(0, 100, 0), 256, 256,
                                            256, None) == -1


def test_strerror():
    lib = B.load_library()
    assert lib.dash_strerror(0) == b"ok"
    for c in (-1, -2, -3, -4, 17):
        assert len(lib.dash_strerror(c)) > 0


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures one GPU; asking for more must end with a message, before anything touches a GPU."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr and r.stdout.strip() == ""


WALK = r"""
#include <cstdio>
#include <vector>
#include "tile_walk.h"
using namespace dash;
// As s2_attend_kernel with two groups of waves: a list of n chunks behind which lies whatever was there, and the mask words
// that the iterations of either group ask for.
int main() {
  int bad = 0;
  for (int n = 0; n <= 40; n++)
    for (int sub_log = 0; sub_log < 2; sub_log++)
      for (int grp = 0; grp < 2; grp++) {
        std::vector<int> list(4096, 0xffff);
        for (int i = 0; i < n << sub_log; i++) list[i] = i;               // the first n chunks, in (n + 31) / 32 mask words
        const ListPart part = list_half(n, grp, sub_log);
        const int n_it = part.chunks << sub_log, words = n > 32 ? 2 : 1;
        auto entry = [&](int i) {
          const int at = walk_index(i, n_it);
          return at < 0 ? 0 : list[(part.first << sub_log) + at];
        };
        int cur = entry(0), next = entry(1), tiles = 0;
        if (part.last_it > 0)
          for (int it = 0; it <= part.last_it; it++) {
            const int u = (cur & 0xfff) >> sub_log, un = (next & 0xfff) >> sub_log;
            if (u >> 5 >= words || un >> 5 >= words) { bad++; std::printf("n %d grp %d it %d: word %d\n", n, grp, it, un >> 5); }
            if (it < n_it && (cur & 0xfff) == (part.first << sub_log) + it) tiles++;
            cur = next;
            next = entry(it + 2);
          }
        if (tiles != n_it) { bad++; std::printf("n %d grp %d: %d tiles of %d\n", n, grp, tiles, n_it); }
      }
  return bad != 0;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no host compiler")
def test_two_groups_read_mask_words_of_their_rows_only(tmp_path):
    """A list of one chunk leaves the second group none; its iterations must not take what lies behind the list for an entry:
    the mask word of such an entry was read up to 127 words past a row."""
    (tmp_path / "walk.cpp").write_text(WALK)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_18753_amd", "csrc"), str(tmp_path / "walk.cpp"), "-o",
                    str(tmp_path / "walk")], check=True, timeout=120)
    r = subprocess.run([str(tmp_path / "walk")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def code_objects(path):
    """The library's gfx950 code objects, as ELF images."""
    blob = open(path, "rb").read()
    for at in (m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob)):
        count, entry = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(count):
            off, size, name_len = struct.unpack_from("<QQQ", blob, entry)
            target = blob[entry + 24:entry + 24 + name_len]
            entry += 24 + name_len
            if b"gfx950" in target:
                yield blob[at + off:at + off + size]


def kernel_scratch(path):
    """Scratch bytes per lane of every kernel: the second word of the kernel's descriptor, which the symbol
    `<kernel>.kd` points at."""
    found = {}
    for elf in code_objects(path):
        sh_off, sh_num = struct.unpack_from("<Q", elf, 40)[0], struct.unpack_from("<H", elf, 60)[0]
        # per section: type, address, file offset, size, linked section
        sections = [struct.unpack_from("<4xI8xQQQI", elf, sh_off + 64 * i) for i in range(sh_num)]
        for kind, _, sym_off, sym_size, link in sections:
            if kind != 11:                                        # dynamic symbols
                continue
            names = sections[link][2]
            for at_sym in range(sym_off, sym_off + sym_size, 24):
                name, index, value = struct.unpack_from("<I2xHQ", elf, at_sym)
                text = elf[names + name:elf.index(b"\0", names + name)].decode()
                if text.endswith(".kd"):
                    _, address, file_off, _, _ = sections[index]
                    found[text[:-3]] = struct.unpack_from("<I", elf, file_off + value - address + 4)[0]
    return found


def test_threshold_solvers_use_no_scratch_memory():
    """The solver that holds four score rows per lane selects one of them by lane; as an indexed load from an array
    that was 32 bytes of scratch in each of these kernels.  Not the builds for rows of more than 512 chunks, whose scores do not
    all fit the registers, nor decode at alpha outside {1.25, 1.5, 2}, where room is set aside that no instruction uses."""
    scratch = kernel_scratch(B.LIB_PATH)
    routing = {n: b for n, b in scratch.items() if re.search(r"14s1_regs_kernelILi\d+ELi\d+ELi\dELi[01]E", n)}
    decode = {n: b for n, b in scratch.items() if re.search(r"16s2_decode_kernelILi\d+ELi0ELi[012]ELb[01]E", n)}
    assert len(routing) == 2 * 5 * 5 * 2 and len(decode) == 2 * 3 * 2
    assert not {n: b for n, b in {**routing, **decode}.items() if b}


def test_prefill_attention_keeps_its_registers():
    """Stage 2 of the prefill holds sums and operands in registers up to what its waves per SIMD leave.  The build with three waves per SIMD spills three of
    them, reloaded where keys are masked, where a maximum rises and behind the tiles; the gathering kernel at head dimension 128 twelve to fifteen, most of
    them reloaded once per item."""
    scratch = kernel_scratch(B.LIB_PATH)
    kernels = {n: b for n, b in scratch.items() if re.search(r"(16s2_attend|16s2_gather|15s2_merge|15s2_costs)_kernel", n)}
    assert len(kernels) == 10 + 8 + 2 + 1
    allowed = {n: 64 if "s2_gather_kernelILi128E" in n else 16 if "s2_attend_kernelILi64ELb0ELb0ELi3E" in n else 0 for n in kernels}
    assert not {n: b for n, b in kernels.items() if b > allowed[n]}


OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WRITES_VECTOR_REGISTERS = re.compile(r"v_(?!writelane|readlane|readfirstlane|cmp)|scratch_|global_|buffer_|flat_|ds_")


def copies_ahead_of_their_lanes(elf_path):
    """Places where a branch that is taken with no lane left lands, or where a loop ends with none left, and vector
    registers are written there before the lanes of the code around it are turned on again."""
    dump = subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", elf_path], stdout=subprocess.PIPE, text=True)
    kernel, start, code, found = None, 0, {}, []

    def check():
        at = sorted(code)
        index = {a: i for i, a in enumerate(at)}
        lands = lambda branch: {start + int(m.group(1), 16) for t in code.values() if t.startswith(branch)
                                for m in [re.search(r"\+0x([0-9a-f]+)>", t)] if m}
        blocks = lands(("s_branch", "s_cbranch"))
        ends = {b for a, b in zip(at, at[1:]) if code[a].startswith("s_cbranch_execnz")}
        for target in (lands("s_cbranch_execz") | ends) & index.keys():
            written = None
            for a in at[index[target]:]:
                text = code[a]
                if a != target and a in blocks:
                    break
                if text.startswith("s_or_b64 exec, exec,"):
                    if written:
                        found.append((kernel, hex(a - start), written))
                    break
                if "exec" in text or text.startswith(("s_branch", "s_endpgm", "s_setpc")):
                    break
                if WRITES_VECTOR_REGISTERS.match(text):
                    written = written or text.split("//")[0].strip()

    for line in dump.stdout:
        if line.endswith(">:\n"):
            if code:
                check()
            address, kernel = line.split(" ", 1)
            start, code = int(address, 16), {}
        elif "//" in line:
            code[int(line.split("//")[1].split(":")[0], 16)] = line.strip()
    if code:
        check()
    assert dump.wait() == 0
    return found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_no_vector_register_is_written_ahead_of_its_lanes(tmp_path):
    """Where many scalar registers are spilled, the compiler can place a copy of a vector register between the spills and the
    instruction that turns the lanes of a branch on again: the copy then reaches the lanes of the branch only.  The
    routing kernel for rows of 1025 to 1536 chunks at a group of 1 was built that way, and gave wrong lists."""
    paths = []
    for i, elf in enumerate(code_objects(B.LIB_PATH)):
        paths.append(str(tmp_path / f"{i}.elf"))
        open(paths[-1], "wb").write(elf)
    assert paths
    with ThreadPoolExecutor(4) as pool:
        assert [x for found in pool.map(copies_ahead_of_their_lanes, paths) for x in found] == []

"""CPU-side checks of the C ABI: the library loads, exports every symbol the
header declares, struct layouts match, and configuration errors are reported
without touching a GPU."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    import torch  # noqa: F401  (HIP runtime first)
    from paper_2512_10576_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2512_10576_amd import build
        build.build()
    return binding.load()


def _declared():
    text = open(os.path.join(ROOT, "include", "ess.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ess_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = _declared()
    assert {"ess_index_score", "ess_topk", "ess_gather_latent", "ess_sparse_mla_decode", "ess_decode_step"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n


def test_struct_layouts():
    from paper_2512_10576_amd import binding as b
    assert C.sizeof(b.EssConfig) == 13 * 4
    assert C.sizeof(b.EssCache) == 5 * 8
    assert C.sizeof(b.EssStats) == 4 * 8
    assert b.EssStepArgs.B.offset == 48 and b.EssStepArgs.idx_out.offset == 64 and C.sizeof(b.EssStepArgs) == 112 and b.EssStepArgs.block_table.offset == 96


def test_config_validation_reports_errors(lib):
    from paper_2512_10576_amd import binding as b
    good = b.make_config(64, 1, 131072, 64, 128, 2048, 128, slots_per_seq=13108)
    n = b.workspace_bytes(good)
    assert n > 64 * 131072 * 4
    cases = [
        (dict(idx_dim=96), b.ESS_ERR_UNSUPPORTED),
        (dict(max_q_tokens=5), b.ESS_ERR_UNSUPPORTED),
        (dict(slots_per_seq=1000), b.ESS_ERR_CAPACITY),
        (dict(row_stride=1150), b.ESS_ERR_INVALID_ARG),
        (dict(max_ctx=1 << 20), b.ESS_ERR_INVALID_ARG),
        (dict(topk=0), b.ESS_ERR_INVALID_ARG),
        (dict(attn_heads=129), b.ESS_ERR_UNSUPPORTED),
    ]
    for change, code in cases:
        kw = dict(max_batch=64, max_q_tokens=1, max_ctx=131072, idx_heads=64, idx_dim=128, topk=2048,
                  attn_heads=128, slots_per_seq=13108)
        kw.update(change)
        with pytest.raises(b.EssError) as ei:
            b.workspace_bytes(b.make_config(**kw))
        assert ei.value.code == code and str(ei.value)
    bad = b.make_config(1, 1, 64, 4, 32, 8, 8)
    bad.struct_size = 8
    with pytest.raises(b.EssError):
        b.workspace_bytes(bad)


@pytest.mark.parametrize("rows,parts", [((1, 1), 64), ((1, 2), 128), ((4, 1), 256), ((5, 1), 320), ((16, 1), 320), ((32, 2), 1280)])
def test_workspace_holds_no_more_partial_results_than_rows_can_use(rows, parts):
    """The room for partial attention results (512 fp16 values, a log-sum-exp and a scale per head): at most 64 splits a
    row, 320 in all for few rows, 20 a row for many.  What 64 more heads add to the workspace is 64 times that."""
    from paper_2512_10576_amd import binding as b
    size = [b.workspace_bytes(b.make_config(*rows, 4096, 64, 128, 512, heads)) for heads in (64, 128)]
    assert size[1] - size[0] == parts * 64 * (512 * 2 + 8)


def test_attention_kernel_agprs_are_only_named_by_its_own_asm(tmp_path):
    """k_attn_partial_tr keeps its 256 output accumulators in AGPRs a0..a255 that its own asm statements name, and
    tells the compiler that the whole AGPR file is taken from a claim statement to a release statement.  Checked in
    the ISA the build flags produce, for all four instances: between claim and release no instruction outside an
    asm statement names an AGPR, nothing is spilled to scratch memory, and no asm MFMA has a vector ALU producer
    of one of its VGPR operands within eight wait states."""
    import collections
    import subprocess
    from paper_2512_10576_amd import build
    out = tmp_path / "sparse_mla.s"
    cmd = [build._hipcc(), *build.compile_flags("sparse_mla.hip"), "-S", "--cuda-device-only",
           os.path.join(build.CSRC, "sparse_mla.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    lines = out.read_text().split("\n")
    starts = [i for i, l in enumerate(lines) if re.match(r"^_ZN\S*k_attn_partial_tr\S*:", l)]
    assert len(starts) == 4                      # one instance per entry format and per way of taking work
    num = r"(?:0x[0-9a-f]+|\d+)"               # the asm printer writes larger register numbers in hexadecimal
    agpr = re.compile(r"\ba\d+\b|\ba\[" + num + r"(:" + num + r")?\]")
    for start in starts:
        end = [i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end")][0]
        tail = "\n".join(lines[end:end + 80])
        assert re.search(r"; ScratchSize: 0\b", tail), "the attention kernel spills registers to scratch memory"
        assert re.search(r"; NumAgprs: 256\b", tail)
        in_asm = claimed = False
        own = collections.Counter()
        n_claim = n_release = 0
        body = []                                # (text, inside an asm statement) between claim and release
        for l in lines[start:end]:
            t = l.strip()
            if t.startswith(";;#ASMSTART"):
                in_asm = True
                continue
            if t.startswith(";;#ASMEND"):
                in_asm = False
                continue
            if in_asm and "ess_agpr_claim" in t:
                claimed, n_claim = True, n_claim + 1
            if in_asm and "ess_agpr_release" in t:
                claimed, n_release = False, n_release + 1
            if not t or t.startswith((";", ".")):
                continue
            if claimed:
                body.append((t, in_asm))
            if agpr.search(t):
                if in_asm:
                    own[t.split()[0]] += 1
                    if t.startswith("v_mfma"):  # accumulate in place: a[x:y], v, v, a[x:y]
                        assert re.search(r"a\[(%s):(%s)\], v\[\d+:\d+\], v\[\d+:\d+\], a\[\1:\2\]" % (num, num), t), t
                else:
                    assert not claimed, "the compiler uses an AGPR of its own where the kernel holds its accumulators: " + t
        assert n_claim >= 1 and n_claim == n_release
        # in every copy of the tile loop the 32 accumulating MFMAs; 256 zero writes, 256 rescale writes and reads per
        # rescale site, 256 final reads
        assert own["v_mfma_f32_32x32x16_bf16"] % 32 == 0 and own["v_mfma_f32_32x32x16_bf16"] >= 32, own
        assert own["v_accvgpr_write_b32"] >= 512 and own["v_accvgpr_read_b32"] >= 512, own
        # hazards of the asm MFMAs (the compiler's hazard logic does not see inside asm statements)
        texts = [t for t, _ in body]
        for i, (t, inside) in enumerate(body):
            m = re.match(r"v_mfma\S* a\[%s:%s\], v\[(\d+):(\d+)\], v\[(\d+):(\d+)\], a\[" % (num, num), t)
            if not (inside and m):
                continue
            used = set(range(int(m[1]), int(m[2]) + 1)) | set(range(int(m[3]), int(m[4]) + 1))
            states = 0
            for prev in reversed(texts[max(0, i - 8):i]):
                if prev.startswith("s_nop"):
                    states += int(prev.split()[1]) + 1
                    continue
                states += 1
                if states > 8 or not prev.startswith("v_") or prev.startswith("v_mfma"):
                    continue
                dst = re.match(r"v_\S+ v(?:\[(\d+):(\d+)\]|(\d+))", prev)
                if dst:
                    wr = set(range(int(dst[1]), int(dst[2]) + 1)) if dst[1] else {int(dst[3])}
                    assert not (wr & used), (prev, t)


def test_topk_kernels_do_not_spill(tmp_path):
    """No form of the top-k but the one that can recompute scores (MODE 3) spills registers to scratch memory, whether
    it takes its rows by workgroup index or by ticket; read from the ISA the build flags produce."""
    import subprocess
    from paper_2512_10576_amd import build
    out = tmp_path / "topk.s"
    subprocess.run([build._hipcc(), *build.compile_flags("topk.hip"), "-S", "--cuda-device-only",
                    os.path.join(build.CSRC, "topk.hip"), "-o", str(out)],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    found = dict(((int(m[1]), m[2] == "1"), int(m[3])) for m in re.finditer(
        r"^_ZN\S*k_topkILi(\d)ELb([01])E\S*:.*?; ScratchSize: (\d+)", out.read_text(), re.S | re.M))
    assert {mode for mode, _ in found} >= {0, 1, 2, 3} and len(found) % 2 == 0
    spills = {form: n for form, n in found.items() if form[0] != 3 and n}
    assert not spills, spills


def _isa(tmp_path, source):
    import subprocess
    from paper_2512_10576_amd import build
    out = tmp_path / source.replace(".hip", ".s")
    subprocess.run([build._hipcc(), *build.compile_flags(source), "-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", str(out)],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return out.read_text().split("\n")


def _sgprs(operand):
    m = re.match(r"s\[(0x[0-9a-f]+|\d+):(0x[0-9a-f]+|\d+)\]$", operand)
    if m:
        return set(range(int(m[1], 0), int(m[2], 0) + 1))
    m = re.match(r"s(\d+)$", operand)
    return {int(m[1])} if m else set()


def _wait_states_before_gathers(lines, start, end):
    """For every memory instruction inside an asm statement that reads scalar registers: the wait states between the last
    vector ALU instruction in front of it that wrote one of them and the instruction (None: none within 40)."""
    body, in_asm, got = [], False, []
    for l in lines[start:end]:
        t = l.strip()
        if t.startswith((";;#ASMSTART", ";;#ASMEND")):
            in_asm = t.startswith(";;#ASMSTART")
            continue
        t = t.split(";")[0].strip()
        if not t or t.startswith(".") or t.endswith(":"):
            continue
        if in_asm and re.match(r"(global|buffer)_", t):
            used = set().union(*(_sgprs(o.split()[0]) for o in t.split(None, 1)[1].split(", ")))
            states, found = 0, None
            for prev in reversed(body[-40:]):
                name, ops = (prev.split(None, 1) + [""])[:2]
                ops = ops.split(", ")
                if name == "s_nop":
                    states += int(ops[0]) + 1
                    continue
                written = _sgprs(ops[0]) | (_sgprs(ops[1]) if re.search("_co_|_u64_u32|_i64_i32|div_scale", name) else set())
                if name.startswith("v_") and written & used:
                    found = states
                    break
                states += 1
            if used:
                got.append((found, body[-6:] + [t]))
        body.append(t)
    return got


@pytest.mark.parametrize("source,kernel", [("sparse_mla.hip", "k_attn_partial_tr"), ("sparse_mla_h32.hip", "k_attn_h32")])
def test_gathers_wait_for_their_scalar_addresses(tmp_path, source, kernel):
    """A memory instruction may read a scalar register that a vector ALU instruction (v_readlane) wrote only five wait states
    later.  The compiler sees to that, but not inside asm statements, which the gathers of the attention kernels are.  Checked
    in the ISA of all instances; also: no instance spills registers to scratch memory."""
    lines = _isa(tmp_path, source)
    starts = [i for i, l in enumerate(lines) if re.match(r"^_ZN\S*%s\S*:" % kernel, l)]
    assert len(starts) == 4                      # one instance per entry format and per way of taking work
    for start in starts:
        end = [i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end")][0]
        assert re.search(r"; ScratchSize: 0\b", "\n".join(lines[end:end + 80])), "the attention kernel spills registers to scratch memory"
        gathers = _wait_states_before_gathers(lines, start, end)
        assert len(gathers) >= 16
        for states, text in gathers:
            assert states is None or states >= 5, "\n".join(text)


def test_short_index_chunks_only_where_they_fit_the_chip_at_once(tmp_path):
    """The index score takes 512 tokens a workgroup only where that makes no more than one workgroup per CU (250 sequences of
    520 tokens would be 500, half of them with 8 tokens); 1024 or, from 2M keys on, 2048 otherwise.  The rule itself,
    compiled for the host."""
    import subprocess
    from paper_2512_10576_amd import build
    shapes = [(1, 1), (1, 8192), (1, 131072), (1, 131073), (2, 65536), (4, 131072), (250, 520), (256, 512), (256, 513), (257, 512), (128, 520),
              (4096, 20), (255, 1), (16, 131072), (13, 131072), (40, 102400), (3, 43691)]
    src = tmp_path / "chunk.hip"
    src.write_text('#include "index_kernel.h"\n#include <stdio.h>\nint main() {\n' + "".join(
        '  printf("%%d\\n", ess_idx::pick_chunk(%d, %d));\n' % s for s in shapes) + "}\n")
    exe = tmp_path / "chunk"
    subprocess.run([build._hipcc(), *build.FLAGS, "-I" + build.CSRC, str(src), "-o", str(exe)], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    got = [int(x) for x in subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE, text=True).stdout.split()]
    for (B, L), chunk in zip(shapes, got):
        want = 512 if B * -(-L // 512) <= 256 else (2048 if B * L >= 2048 * 1024 else 1024)
        assert chunk == want, (B, L, chunk)


def test_append_to_flat_keys_hands_no_scale_array_to_the_kernel(lib, tmp_path):
    """Only a paged Indexer-Cache has key scales: with flat keys ess_append takes whatever new_key_scale holds, and the kernel
    must not read it.  What the launch passes is taken from the runtime's launch functions, replaced in a process of its own (no GPU)."""
    import subprocess
    import sys
    (tmp_path / "shim.c").write_text(
        "#include <stddef.h>\n"
        "typedef struct { unsigned x, y, z; } d3;\n"
        "void* shim_seen; int shim_launches;\n"
        "int __hipPushCallConfiguration(d3 g, d3 b, size_t lds, void* st) { return 0; }\n"
        "int __hipPopCallConfiguration(d3* g, d3* b, size_t* lds, void** st) {\n"
        "  d3 one = {1, 1, 1}; *g = one; *b = one; *lds = 0; *st = 0; return 0;\n}\n"
        "int hipLaunchKernel(const void* f, d3 g, d3 b, void** args, size_t lds, void* st) {\n"
        "  shim_seen = *(void**)args[16]; ++shim_launches; return 0;\n}\n")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(tmp_path / "shim.so"), str(tmp_path / "shim.c")], check=True)
    (tmp_path / "run.py").write_text("""
import ctypes as C, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
import torch
from paper_2512_10576_amd import binding as b
lib = b.load()
cfg = b.make_config(1, 1, 256, 4, 32, 8, 8)
cache = b.EssCache(4096, None, 4096, 4096, 4096)
f = lib._Z17ess_launch_appendRK10ess_configRK9ess_cachePKhS6_PhPiiijS8_PKfPKiiP12ihipStream_t
vp, i32 = C.c_void_p, C.c_int32
f.argtypes = [vp, vp, vp, vp, vp, vp, i32, i32, C.c_uint32, vp, vp, vp, i32, vp]
for table, want in ((None, None), (4096, 0x1234)):
    f(C.addressof(cfg), C.addressof(cache), 4096, 4096, 4096, 4096, 1, 1, 1, None, 0x1234, table, 1, None)
    got = C.c_void_p.in_dll(shim, "shim_seen").value
    assert got == want, (table, got)
assert C.c_int.in_dll(shim, "shim_launches").value == 2
print("handed over as it should be")
""")
    p = subprocess.run([sys.executable, str(tmp_path / "run.py"), str(tmp_path / "shim.so")], cwd=ROOT, stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True, env=dict(os.environ, PYTHONPATH=ROOT))
    assert p.returncode == 0 and "handed over as it should be" in p.stdout, p.stdout


def test_whole_rows_narrow_to_the_digit_of_the_kth_score(tmp_path):
    """A row held whole is spread evenly over digits, and the keys of the digit that holds the k-th largest score again among
    themselves, until counting can take what is left or it is equal.  The spread itself, compiled for the host and replayed from the row's
    extremes: rows as they come need no second round, one outlier or a mask of the lowest number one, both two, magnitudes apart
    three at most, and none ends in the general selection (-1)."""
    import subprocess
    import numpy as np
    from paper_2512_10576_amd import build
    src = tmp_path / "narrow.hip"
    src.write_text('''#include "select_common.h"
#include <stdio.h>
#include <cmath>
#include <vector>
using namespace ess_sel;
int main(int argc, char** argv) {
  const int n = atoi(argv[2]), k = atoi(argv[3]);
  std::vector<float> row(n);
  FILE* f = fopen(argv[1], "rb");
  while (fread(row.data(), 4, n, f) == (size_t)n) {
    float lo = INFINITY, hi = -INFINITY;
    for (float x : row) if (std::isfinite(x)) { lo = fminf(lo, x); hi = fmaxf(hi, x); }
    std::vector<float> v = row;                      // the keys still in question
    int take = k, rounds = -1;
    for (int round = 0; round <= NARROW; ++round) {
      const Spread sp(lo, hi);
      if (round > 0 && lo == hi) { rounds = round; break; }          // equal: by position
      if (round > 0 && sp.scale == 0.f) break;
      std::vector<std::vector<float>> h(NBINS);
      for (float x : v)
        h[sp.scale != 0.f ? sp.digit(x) : (x == INFINITY ? NBINS - 1 : (x > -INFINITY ? 1u : 0u))].push_back(x);
      float top = -INFINITY;                                         // the digits keep the order of the scores
      for (auto& part : h) {
        for (float x : part) if (x < top) { printf("disorder\\n"); return 1; }
        for (float x : part) top = fmaxf(top, x);
      }
      int at = NBINS - 1;
      while (take > (int)h[at].size()) take -= (int)h[at--].size();
      v = h[at];
      if (v.size() <= FEW || (int)v.size() == take) { rounds = round; break; }
      lo = INFINITY; hi = -INFINITY;
      for (float x : v) { const float y = x == x ? x : -INFINITY; lo = fminf(lo, y); hi = fmaxf(hi, y); }
    }
    printf("%d\\n", rounds);
  }
}
''')
    n, k = 8000, 2048
    rng = np.random.RandomState(3)
    base = (rng.randn(n) * 40 + 300).astype(np.float32)

    def with_(at, value, x=base):
        x = x.copy()
        x[at] = value
        return x

    mask = with_(slice(0, n, 5), -3.4028235e38)
    rows = [(base, 0, 0), (with_([5], 300 + 40 * 50), 0, 0), (with_([5], 300 + 40 * 1000), 1, 1), (with_([5], 1e30), 1, 1),
            (with_([5], -1e30), 1, 1), (mask, 1, 1), (with_([7], 1e30, mask), 1, 2), (with_([7], 3.4028235e38, with_([8], -3.4028235e38)), 1, 1),
            (with_(slice(0, n, 7), -np.inf), 0, 0), (with_([7, 9, 11], [1e30, np.inf, np.nan], with_(slice(0, n, 5), -np.inf)), 1, 1),
            (np.exp((base - 300) / 20).astype(np.float32), 1, 3), (np.exp((base - 300) / 10).astype(np.float32), 1, 3),
            (with_(slice(0, n, 20), np.sort(base)[-k]), 1, 2), (with_(slice(0, n), 2.5), 1, 1), (with_(slice(0, n, 2), np.sort(base)[-k]), 1, 2),
            (np.where(rng.rand(n) < 0.1, np.float32(7.0), np.float32(7.000001)), 0, 1), (with_(slice(0, n), np.nan), 1, 1),
            (with_(slice(100, n), -np.inf, with_(slice(0, n, 3), np.nan)), 1, 1)]
    np.stack([r[0] for r in rows]).astype(np.float32).tofile(tmp_path / "rows")
    exe = tmp_path / "narrow"
    subprocess.run([build._hipcc(), *build.FLAGS, "-I" + build.CSRC, str(src), "-o", str(exe)], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    got = [int(x) for x in subprocess.run([str(exe), str(tmp_path / "rows"), str(n), str(k)], check=True, stdout=subprocess.PIPE, text=True).stdout.split()]
    assert len(got) == len(rows)
    for i, (rounds, (_, least, most)) in enumerate(zip(got, rows)):
        assert least <= rounds <= most, (i, rounds)


def test_sample_target_leaves_room_on_both_sides(tmp_path):
    """The list of a sampled row takes what reaches the t-th largest of its samples: it must hold the k largest and fit its buffer.  For every k and row
    length the bound has to be one the list can be made with (it once asked for more than fits for k above 3500 past 131072 positions), and both
    ways of missing must be rare where samples are drawn at random."""
    import subprocess
    from scipy.stats import hypergeom
    from paper_2512_10576_amd import build
    cap, shapes = 8192, []
    for vis in (8193, 8224, 12000, 20000, 40000, 65536, 115000, 131072, 131088, 140000, 200000, 262144, 262160, 300000, 400001, 524288):
        blocks = vis >> 4                                # the sample, as the kernel takes it
        for k in (1, 2, 16, 100, 513, 1024, 2048, 3000, 3584, 4000, 4096):
            most, stride = 512 if k > 2048 and vis > 262144 else 256, 1
            while blocks // stride > most:
                stride <<= 1
            shapes.append((k, blocks // stride << 4, vis))
        shapes += [(k, -(-vis // 32) // 64 * 64, vis) for k in (1, 513, 2048, 4096) if vis <= 262144]      # and of the fused selection
    src = tmp_path / "target.hip"
    src.write_text('#include "select_common.h"\n#include <stdio.h>\nint main(int c, char** v) {\n'
                   "  for (int i = 1; i + 2 < c; i += 3)\n"
                   '    printf("%u\\n", ess_sel::sample_target(atoi(v[i]), (float)atoi(v[i + 1]) / atoi(v[i + 2])));\n}\n')
    exe = tmp_path / "target"
    subprocess.run([build._hipcc(), *build.FLAGS, "-I" + build.CSRC, str(src), "-o", str(exe)], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    got = subprocess.run([str(exe), *(str(x) for s in shapes for x in s)], check=True, stdout=subprocess.PIPE, text=True).stdout.split()
    assert len(got) == len(shapes)
    for (k, ns, vis), t in zip(shapes, map(int, got)):
        assert 1 <= t and t * vis < 0.85 * cap * ns, (k, ns, vis, t)
        short = hypergeom.sf(t - 1, vis, k, ns)          # t or more of the samples among the k largest
        full = hypergeom.cdf(t - 1, vis, cap, ns)        # fewer than t among those that fit
        assert short + full < 2e-3, (k, ns, vis, t, short, full)

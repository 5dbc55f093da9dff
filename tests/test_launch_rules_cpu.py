"""The rules that choose kernels: the compile-time ones read from the headers by
a host program, the library's own called from one."""
import os
import subprocess

from paper_2603_28770_amd import build as B
from paper_2603_28770_amd import user_objectives as U

OBJ = {"rosenbrock": 0, "rastrigin": 1, "ackley": 2, "styblinski_tang": 3, "goldstein_price": 4,
       "sphere": 5, "quartic": 6}


def _host_program(tmp_path, headers, body):
    src = tmp_path / "rule.hip"
    src.write_text("".join(f'#include "{h}"\n' for h in headers) + "#include <stdio.h>\n"
                   "using namespace zeus;\nint main() {\n" + body + "\nreturn 0;\n}\n")
    exe = tmp_path / "rule"
    r = subprocess.run([B._hipcc(), "--offload-host-only", "-std=c++17", "-O0", "-w", "-I", B.CSRC,
                        "-x", "hip", str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout


def test_lanes_are_shared_where_starts_stall(tmp_path):
    # not where the minimum is zero (no start stalls), not by a whole wave (no
    # other group), and by two groups of 32 lanes only where it pays
    body = "".join(f'printf("{name} {g} %d\\n", (int)kShareLanes<{o}, {g}>);\n'
                   for name, o in OBJ.items() for g in (2, 4, 8, 16, 32, 64))
    got = {tuple(l.split()[:2]): l.split()[2] == "1"
           for l in _host_program(tmp_path, ["zeus_bfgs_common.h"], body).splitlines()}
    for name in OBJ:
        for g in (2, 4, 8, 16, 32, 64):
            stalls = name in ("rastrigin", "ackley", "styblinski_tang", "goldstein_price")
            want = stalls and g < 64 and not (g == 32 and name == "styblinski_tang")
            assert got[name, str(g)] == want, (name, g)


def test_user_code_shares_no_lanes_at_32(tmp_path):
    # a whole-form objective tries one length per lane: 32 lanes reach past the
    # last trial of a search by themselves
    (tmp_path / "user.h").write_text('#include "zeus_user.h"\n' + U.ROSENBROCK)
    body = 'printf("%d %d %d\\n", kShareLanes<kUser, 16>, kShareLanes<kUser, 32>, kShareLanes<kUser, 64>);'
    out = _host_program(tmp_path, [str(tmp_path / "user.h"), "zeus_user_elem.h", "zeus_bfgs_common.h"],
                        body)
    assert out.split() == ["1", "0", "0"]


def _library_program(tmp_path, code, stdin):
    """Output lines of a program that calls the library's own rules."""
    from paper_2603_28770_amd import zeus as Z
    (tmp_path / "rule.cpp").write_text('#include "zeus_internal.h"\n#include <stdio.h>\n'
                                       "int main() {\n" + code + "\nreturn 0; }\n")
    exe = tmp_path / "rule"
    r = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w", "-I", B.CSRC, "-I",
                        "/opt/rocm/include", str(tmp_path / "rule.cpp"), Z.LIB_PATH,
                        f"-Wl,-rpath,{os.path.dirname(Z.LIB_PATH)}", "-L/opt/rocm/lib",
                        "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64", "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return subprocess.run([str(exe)], input=stdin, capture_output=True, text=True,
                          check=True).stdout.split()


def test_lbfgs_kernel_of_a_launch(tmp_path):
    # few starts, and in mixed precision the objectives whose starts stall, take
    # a coordinate per lane
    cases = [(o, p, s, n) for o in OBJ.values() for p in (0, 1) for s in (8, 16, 32, 64, 128)
             for n in (1, 256, 1024, 4096, 4097, 65536, 2**40)]
    out = _library_program(
        tmp_path, 'int o, p, s; long n;\nwhile (scanf("%d %d %d %ld", &o, &p, &s, &n) == 4)\n'
        '  printf("%d\\n", (int)zeus::lbfgs_spread(o, p, s, n, 12288 * 16 / s, 256));',
        "".join("%d %d %d %d\n" % c for c in cases))
    assert len(out) == len(cases)
    for (o, p, s, n), got in zip(cases, out):
        lanes = n * min(s, 64)
        if s == 8 and o != OBJ["rosenbrock"]:
            want = lanes <= 32768  # half a wavefront on each SIMD of 256 units
        else:
            want = n <= 12288 * 16 // s and lanes <= 3 * 65536
            if p == 1:
                want = want or o in (OBJ["rastrigin"], OBJ["styblinski_tang"]) or (o == OBJ["ackley"] and s == 16)
        assert (got == "1") == want, (o, p, s, n)


def test_three_wavefront_blocks(tmp_path):
    # with the transcendental terms only launches of more than eight starts per
    # unit, in mixed precision sixteen (they are slower one by one, and more of
    # them fit)
    cases = [(o, p, n) for o in OBJ.values() for p in (0, 1) for n in (1, 512, 2048, 2049, 4096, 4097, 65536)]
    out = _library_program(
        tmp_path, 'int o, p; long n;\nwhile (scanf("%d %d %ld", &o, &p, &n) == 3)\n'
        '  printf("%d\\n", (int)zeus::tile_three(o, p, n, 256));',
        "".join("%d %d %d\n" % c for c in cases))
    assert len(out) == len(cases)
    for (o, p, n), got in zip(cases, out):
        costly = o in (OBJ["rastrigin"], OBJ["ackley"])
        assert (got == "1") == (not costly or n > (4096 if p else 2048)), (o, p, n)


def test_wide_slots(tmp_path):
    # the least slot holds the strips that the wide block keeps there (its second
    # tile's columns from 160 on, two strips of 16 columns by 512 rows), no launch
    # needs more than the public sizes count, and a server step of 64 MiB has a
    # slot for every unit
    code = ('for (int d = 1; d <= 256; ++d)\n  for (long n : {1l, 300l, 5000l})\n'
            '    printf("%d %ld %d %ld %ld %zu %zu\\n", d, n, zeus::wide_slots(n),\n'
            '           (long)zeus::wide_slot_doubles(d), (long)zeus::wide_slot_least(d),\n'
            '           zeus::wide_hslot_bytes(n, d), zeus::wide_reserved_bytes(n, d));')
    vals = [int(v) for v in _library_program(tmp_path, code, "")]
    rows = [vals[i:i + 7] for i in range(0, len(vals), 7)]
    assert len(rows) == 256 * 3
    for d, n, slots, apart, least, need, reserved in rows:
        assert slots == min(n, 256) and least <= apart and need == 8 * slots * apart
        assert apart % 2 == 0 and least % 2 == 0
        assert need <= reserved == 8 * min(n, 2048) * d * ((d + 63) // 64 * 64)
        if d > 160:
            assert least == 16 * 1024 and (64 << 20) // (8 * least) >= 256


def test_autotuner_times_what_a_table_entry_runs(tmp_path):
    # an entry of 64 lanes runs the cut tile where there is one (the library's own
    # choice for every objective and dimension that the table gives 64 lanes)
    from paper_2603_28770_amd import autotune as A
    cases = [(name, prec, d) for name in A.OBJECTIVES for prec in (0, 1) for d in range(33, 65)]
    out = _library_program(
        tmp_path, 'int o, p, d;\nwhile (scanf("%d %d %d", &o, &p, &d) == 3)\n'
        '  printf("%d\\n", zeus::group_lanes(o, p, d));',
        "".join("%d %d %d\n" % (A.OBJECTIVES[n], p, d) for n, p, d in cases))
    for (name, prec, d), got in zip(cases, out):
        assert int(got) == A.forced_tiling(name, d, 64), (name, prec, d)
    assert A.forced_tiling("rosenbrock", 40, 256) == 256 and A.forced_tiling("rosenbrock", 16, 16) == 16

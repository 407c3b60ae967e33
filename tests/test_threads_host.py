"""Cases of one mesh planned on several threads at once: the structures a mesh
builds on first use (parts of the resident solves, AMG hierarchy) are built
once and without a data race.

The host sources are rebuilt by the system compiler under ThreadSanitizer
into a small program (the HIP kernels' object is linked unchanged; nothing
here launches a kernel).
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1207_1571_amd", "csrc")
KERNELS_OBJ = os.path.join(ROOT, "paper_1207_1571_amd", "_build", "kernels.o")

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>
#include "fvm.h"

// a box of n^3 unit cells
static fvm_mesh *box(int n)
{
    std::vector<int32_t> own, nei;
    std::vector<double> S, Cf, C, V((size_t)n * n * n, 1.0);
    std::vector<int32_t> bown;
    std::vector<double> bS, bCf;
    auto id = [n](int i, int j, int k) { return (k * n + j) * n + i; };
    for (int k = 0; k < n; ++k)
        for (int j = 0; j < n; ++j)
            for (int i = 0; i < n; ++i) {
                const int x[3] = {i, j, k};
                for (int a = 0; a < 3; ++a) C.push_back(x[a] + 0.5);
                for (int a = 0; a < 3; ++a)
                    for (int s = -1; s <= 1; s += 2) {
                        const bool inside = s < 0 ? x[a] > 0 : x[a] + 1 < n;
                        if (inside && s < 0) continue;
                        std::vector<double> &vs = inside ? S : bS, &vc = inside ? Cf : bCf;
                        for (int b = 0; b < 3; ++b) {
                            vs.push_back(b == a ? s : 0.0);
                            vc.push_back(x[b] + (b == a ? (s > 0 ? 1.0 : 0.0) : 0.5));
                        }
                        if (inside) {
                            own.push_back(id(i, j, k));
                            nei.push_back(id(i + (a == 0), j + (a == 1), k + (a == 2)));
                        } else bown.push_back(id(i, j, k));
                    }
            }
    const int32_t Fi = (int32_t)own.size(), Fb = (int32_t)bown.size();
    own.insert(own.end(), bown.begin(), bown.end());
    S.insert(S.end(), bS.begin(), bS.end());
    Cf.insert(Cf.end(), bCf.begin(), bCf.end());
    fvm_patch p;
    std::memset(&p, 0, sizeof(p));
    p.start = Fi; p.size = Fb; p.u_kind = FVM_BC_FIXED; p.p_kind = FVM_BC_ZERO_GRAD;
    const fvm_mesh_desc d = {n * n * n, Fi + Fb, Fi, 1, own.data(), nei.data(), S.data(), Cf.data(), C.data(), V.data(), &p};
    fvm_mesh *m = nullptr;
    if (fvm_mesh_create(&d, &m) != FVM_OK) std::printf("mesh: %s\n", fvm_last_error());
    return m;
}

int main()
{
    fvm_case_opts o;
    std::memset(&o, 0, sizeof(o));
    o.nu = 0.1; o.dt = 0.1; o.alpha_u = o.alpha_p = 1.0; o.inner_rel_tol = 1e-3; o.inner_max_iter = 10; o.n_corr = 2;
    o.p_ctl.tol = o.u_ctl.tol = 1e-6;
    o.p_ctl.max_iter = o.u_ctl.max_iter = 10;
    // every kind of structure: FP64 Jacobi, DIC and AMG cases, mixed ones
    for (int kind = 0; kind < 4; ++kind) {
        fvm_mesh *m = box(20);
        if (!m) return 1;
        o.p_ctl.precond = kind == 3 ? 0 : kind;
        o.precision = kind == 3 ? FVM_MIXED : FVM_FP64;
        size_t bytes[4] = {0, 0, 0, 0};
        fvm_status st[4];
        std::vector<std::thread> ts;
        for (int t = 0; t < 4; ++t)
            ts.emplace_back([&, t] { st[t] = fvm_case_workspace_bytes(m, &o, &bytes[t]); });
        for (auto &t : ts) t.join();
        for (int t = 0; t < 4; ++t)
            if (st[t] != FVM_OK || bytes[t] == 0 || bytes[t] != bytes[0]) return 2;
        fvm_mesh_destroy(m);
    }
    std::printf("planned\n");
    return 0;
}
"""


def test_cases_of_one_mesh_on_several_threads(tmp_path):
    if not os.path.exists(KERNELS_OBJ):
        pytest.skip("libfvm has not been built (no kernels object to link)")
    rt = subprocess.check_output(["gcc", "-print-file-name=libtsan.so"], text=True).strip()
    if not os.path.isabs(rt):
        pytest.skip("sanitizer runtime not available")
    (tmp_path / "main.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "plan")
    subprocess.check_call(
        ["g++", "-std=c++17", "-fsanitize=thread", "-g", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
         os.path.join(ROOT, "include"), "-I", CSRC, str(tmp_path / "main.cpp"), os.path.join(CSRC, "mesh.cpp"),
         os.path.join(CSRC, "case.cpp"), KERNELS_OBJ, "-o", exe, "-pthread", "-L/opt/rocm/lib", "-lamdhip64",
         "-lrocprofiler-sdk-roctx", "-Wl,-rpath,/opt/rocm/lib"])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=dict(os.environ, TSAN_OPTIONS="halt_on_error=0"))
    if "unexpected memory mapping" in r.stderr:
        pytest.skip("ThreadSanitizer does not run under this kernel's address layout")
    assert "planned" in r.stdout, (r.returncode, r.stdout, r.stderr[-2000:])
    ours = re.findall(r"data race[^\n]*(?:\n(?!==).*)*", r.stderr)
    ours = [x for x in ours if "mesh.cpp" in x or "case.cpp" in x]
    assert not ours, ours[0][:3000]

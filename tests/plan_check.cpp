// Checks of a plan whose panels live in LDS, against the front tree that it was built
// from: what the solver's kernels read without a bounds check of their own.
//   plan_check NDIM N BC LEAF WAVE_MAX_M   ("panels", "global", or the first violation)
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <stdexcept>
#include <string>
#include <vector>

#include "../paper_1908_08292_amd/csrc/plan.h"

using namespace fehmm;

namespace {

void need(bool ok, const std::string& what, int a = -1, int b = -1) {
    if (ok) return;
    std::printf("%s (%d, %d)\n", what.c_str(), a, b);
    std::exit(1);
}

int64_t cpk(int64_t j, int64_t m) { return j * m - j * (j - 1) / 2; }

}  // namespace

int main(int argc, char** argv) {
    if (argc != 6) return 2;
    const int d = std::atoi(argv[1]), n = std::atoi(argv[2]);
    PlanParams pp;
    pp.bc = std::atoi(argv[3]);
    pp.leaf = std::atoi(argv[4]);
    pp.wave_max_m = std::atoi(argv[5]);
    const PlanHost P = build_plan(d, n, pp);
    if (!P.panel_path) {
        std::printf("global\n");
        return 0;
    }
    const int ns = (int)P.fronts.size();
    const int64_t rc = d * d + (d == 2 ? 1 : 0);  // right-hand-side columns at most
    need(P.lds_path || P.wide_rhs, "wide_rhs not set");

    // original entries: distinct offsets within the packed panel
    for (int s = 0; s < ns; ++s) {
        const FrontHost& F = P.fronts[s];
        std::set<int> seen;
        for (int t = F.asm_begin; t < F.asm_end; ++t) {
            need(P.asm_dst[t] >= 0 && P.asm_dst[t] < cpk(F.p, F.m), "original entry outside the panel", s, t);
            need(seen.insert(P.asm_dst[t]).second, "original entry stored twice", s, t);
        }
    }

    // inverse row maps and the panel prefix of every update matrix
    for (int s = 0; s < ns; ++s) {
        const FrontHost& F = P.fronts[s];
        if (F.parent < 0) continue;
        const FrontHost& A = P.fronts[F.parent];
        const int mc = F.m - F.p;
        std::vector<int> want(A.m, -1);
        for (int q = 0; q < mc; ++q) {
            const int row = P.relind[F.relind_off + q];
            need(row >= 0 && row < A.m, "child row outside the parent", s, q);
            need(q == 0 || row > P.relind[F.relind_off + q - 1], "child rows out of order", s, q);
            want[row] = (int)((cpk(q, mc) - q) << 16) | q;
        }
        for (int r = 0; r < A.m; ++r) need(P.inv[F.inv_off + r] == want[r], "inverse row map", s, r);
        for (int64_t t = 0; t < cpk(mc, mc); ++t) {
            const int64_t to = P.ea_dst[F.ea_off + t];
            need(to >= 0 && to < cpk(A.m, A.m), "extend-add target", s, (int)t);
            need((to < cpk(A.p, A.m)) == (t < F.npre), "prefix of the update matrix in the parent's panel", s, (int)t);
        }
    }

    // wave tasks: every wave front once, after its children
    std::vector<int> task_of(ns, -1), level_of(ns, -1);
    const int nlev = (int)P.task_beg.size() - 1;
    for (int h = 0; h < nlev; ++h)
        for (int k = P.task_beg[h]; k < P.task_beg[h + 1]; ++k)
            for (int s = P.task[2 * k]; s <= P.task[2 * k + 1]; ++s) {
                need(P.fronts[s].wave && task_of[s] < 0, "task front", s, k);
                task_of[s] = k;
                level_of[s] = h;
                for (int q = P.fronts[s].child_begin; q < P.fronts[s].child_end; ++q) {
                    const int c = P.children[q];
                    need(task_of[c] == k || (task_of[c] >= 0 && level_of[c] < h), "task before its children", s, c);
                }
            }
    bool all_wave = true;
    for (int s = 0; s < ns; ++s) {
        const FrontHost& F = P.fronts[s];
        all_wave = all_wave && F.wave;
        need(!F.wave == (task_of[s] < 0), "wave front without a task", s);
        need(!F.wave || F.m <= 64, "wave front with more rows than lanes", s);
    }

    // LDS of the wave phase: slices, then the update matrices that stay there; for
    // FP64 elements and for FP32 ones with right-hand sides of 8 bytes (wide_rhs)
    for (int es = 4; es <= 8; es += 4) {
        const int64_t rw = P.wide_rhs && es == 4 ? 2 : 1;
        const int64_t block = 2 * 16 * rc * rw + 2;
        for (int s = 0; s < ns; ++s) {
            const FrontHost& F = P.fronts[s];
            if (!F.wave) continue;
            need(cpk(F.p, F.m) + block <= P.wave_slice, "wave slice", s);
            if (F.u_lds < 0) continue;
            need(F.parent >= 0 && (P.ul_stride == 0 || task_of[F.parent] == task_of[s]), "update matrix left in LDS", s);
            need(P.ul_stride > 0 || all_wave, "update matrices shared by the waves", s);
            const int64_t mu = F.m - F.p, tri = (cpk(mu, mu) + rw - 1) / rw * rw, end = F.u_lds + tri + mu * rc * rw;
            need(F.u_lds >= 2 && F.u_lds % rw == 0, "update matrix offset", s);
            need(P.ul_stride > 0 ? end <= P.ul_stride : P.ul_base + end <= P.wave_elems, "update matrix past its room", s);
            for (int q = 0; q < ns; ++q) {
                const FrontHost& G = P.fronts[q];
                if (q == s || G.u_lds < 0 || (P.ul_stride > 0 && task_of[q] != task_of[s])) continue;
                need(G.u_lds >= end || G.u_lds < F.u_lds, "update matrices overlap", s, q);
            }
        }
        // workgroup steps: every other front once, after its children, side by side
        // only with equal barriers, a thread per row, two panels at most in LDS
        std::vector<char> done(ns, 0), once(ns, 0);
        for (int s = 0; s < ns; ++s) done[s] = P.fronts[s].wave ? 1 : 0;
        for (size_t st = 0; st < P.wg_steps.size() / kStepFronts; ++st) {
            std::vector<int> fs;
            for (int k = 0; k < kStepFronts; ++k)
                if (P.wg_steps[kStepFronts * st + k] >= 0) {
                    need((int)fs.size() == k, "step with a gap", (int)st);
                    fs.push_back(P.wg_steps[kStepFronts * st + k]);
                }
            need(fs.size() == 1 || fs.size() == 2 || fs.size() == 4, "step size", (int)st);
            int64_t panel = 0;
            for (int s : fs) {
                const FrontHost& F = P.fronts[s];
                need(!F.wave && !once[s], "step front", (int)st, s);
                once[s] = 1;
                for (int q = F.child_begin; q < F.child_end; ++q) need(done[P.children[q]], "step before its children", s);
                const FrontHost& A = P.fronts[fs[0]];
                need(F.p == A.p && F.child_end - F.child_begin == A.child_end - A.child_begin, "unequal barriers", (int)st, s);
                need(F.m <= (fs.size() == 1 ? 64 * kSolveWaves : 128), "more rows than threads", (int)st, s);
                panel = std::max(panel, cpk(F.p, F.m));
                const int64_t nw = kSolveWaves / (int)fs.size();
                need(rc * (F.m + (F.m > F.p ? nw * F.p : 0)) <= nw * P.bs_slice, "backward substitution scratch", (int)st, s);
            }
            for (int s : fs) done[s] = 1;
            panel = (panel + rw - 1) / rw * rw;
            need(std::min<int>((int)fs.size(), kStepGroups) * (panel + block) <= P.wg_elems, "step past the LDS", (int)st);
        }
        for (int s = 0; s < ns; ++s) need(done[s], "front never factored", s);
    }
    if (P.wave_list.size()) need(P.bs_slice >= 4 * (rc * 64 + 4), "backward substitution scratch of wave fronts");
    const int64_t lds = 8 * std::max<int64_t>({P.wave_elems, P.wg_elems, kSolveWaves * P.bs_slice, P.max_m * rc});
    need(lds + 6 * 1024 + 1024 <= 160 * 1024, "LDS of a workgroup", (int)lds);

    // update matrices in the workspace: disjoint slots behind the zero element
    int64_t at = 2;
    for (int s = 0; s < ns; ++s) {
        const int64_t mu = P.fronts[s].m - P.fronts[s].p;
        need(P.fronts[s].U_off >= at, "update slot", s);
        at = P.fronts[s].U_off + mu * (mu + 1) / 2 + mu * rc + 1;
        need(at <= P.U_stack + (mu == 0 ? 1 : 0), "update slot past the region", s);
    }
    std::printf("panels\n");
    return 0;
}

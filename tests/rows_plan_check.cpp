// Reads cases "vpp B N J_0 .. J_{N-1}" and prints, for the build list and the
// final list of the row form, every workgroup as "list kind first count P" after the
// list's tasks "list k f row-form-key" (see test_rows_plan.py).
#include <cstdio>

#include "swr_rows_plan.h"

using namespace swr;

int main() {
    int vpp, B, N;
    while (std::scanf("%d %d %d", &vpp, &B, &N) == 3) {
        std::vector<int> J(N), Pk(N);
        for (int k = 0; k < N; ++k) {
            if (std::scanf("%d", &J[k]) != 1) return 1;
            Pk[k] = (J[k] + kWave) / kWave;
        }
        const int nv = vpp ? B : 1;
        std::vector<Task> list[2];
        for (int v = 0; v < nv; ++v)
            for (int k = 0; k < N; ++k)
                for (int e = 0; e < 2; ++e)
                    if (e == 0 ? k >= 1 : k <= N - 2) list[0].push_back(Task{k, 0, v * N + k, 0});
        for (int q = 0; q < 2; ++q)
            for (int b = 0; b < B; ++b)
                for (int k = 0; k < N; ++k) list[q].push_back(Task{k, b, (vpp ? b : 0) * N + k, 0});
        const RowsPlan p = rows_plan(J, Pk, list[0].size() + list[1].size(), vpp ? 0 : B);
        for (int q = 0; q < 2; ++q) {
            sort_tasks(list[q], Pk, p.rows);
            RowsList out;
            rows_items(p.rows, list[q], false, out);
            for (const Task& t : list[q]) std::printf("t %d %d %d %d\n", q, t.k, t.f, p.rows[t.k]);
            for (const RowsRun& r : out.runs)
                for (int i = r.start; i < r.start + r.count; ++i)
                    std::printf("w %d %d %d %d %d\n", q, r.kind, out.host[i].x, out.host[i].y, out.host[i].z);
        }
        std::printf("end\n");
    }
    return 0;
}

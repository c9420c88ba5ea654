// swr_rows_plan.h -- host side of the row and wide forms: which form every
// subdomain has, the order of a task list, and the workgroups a list is cut into.
// No GPU calls: plain functions of the problem's sizes.
#pragma once
#include <algorithm>
#include <vector>

#include "swr_common.h"

namespace swr {

// Wide form: waves per task for a subdomain of at most 64 Pk nodes (Pk > kMaxP),
// 0 past its sizes.  More waves than needed for 5 to 9 nodes per lane only add
// exchanges; fewer would not hold the state in registers.
inline int wide_waves(int Pk) { return Pk <= 18 ? 2 : Pk <= 36 ? 4 : Pk <= 8 * kWideMaxP ? 8 : 0; }

// ---------------------------------------------------------------------------
// Row form of the static sweep: how many rows of 16 lanes a task of each
// subdomain gets.  Fewer rows put more tasks in a wave and cost less per task
// (each step's separator reduction, boundary terms and lane moves are shared by
// the wave's tasks), but need more tasks to fill the GPU and more registers
// per lane; wide tasks keep their interior coefficients in LDS, one copy per
// workgroup, which wants tasks that share a record.  The choice depends on
// the problem's sizes only, never on the schedule, so every schedule computes
// the same bits.
// ---------------------------------------------------------------------------
struct RowsPlan {
    std::vector<int> rows;       // P + 32 RW of every subdomain (0: another form)
    std::vector<int> wide;       // P + 32 NW (0: another form)
    size_t rstride = 0, wstride = 0;
    bool streams = false;        // subdomains past the wide form's sizes
};
// J: cells, Pk: nodes per lane of a whole wave; ntasks: tasks that overlap;
// sharing: tasks of a list with one record
inline RowsPlan rows_plan(const std::vector<int>& J, const std::vector<int>& Pk, size_t ntasks, int sharing) {
    RowsPlan p;
    p.rows.assign(J.size(), 0);
    p.wide.assign(J.size(), 0);
    const bool shared = sharing >= 4;
    for (size_t k = 0; k < J.size(); ++k) {
        const int n = J[k] + 1;
        if (n > kWave * kMaxP) {
            const int NW = wide_waves(Pk[k]);
            if (NW == 0) { p.streams = true; continue; }
            const int P = (Pk[k] + NW - 1) / NW;
            p.wide[k] = P + 32 * NW;
            p.wstride = std::max(p.wstride, wide_record(P, NW));
            continue;
        }
        int RW = 4;
        if (n <= 128) {
            if (ntasks >= kRowsFill1) RW = 1;
        } else if (n <= 224 && shared && ntasks >= kRowsFill1Lds) {
            RW = 1;
        } else if (n <= 256) {
            if (ntasks >= kRowsFill2) RW = 2;
        } else if (shared && ntasks >= kRowsFill2Lds) {
            RW = 2;
        }
        const int T = 16 * RW, P = (n + T - 1) / T;
        p.rows[k] = P + 32 * RW;
        p.rstride = std::max(p.rstride, (size_t)rows_fields(P, RW) * T);
    }
    return p;
}

// The order of a task list: width of a whole wave (widest first; the launches by
// width take runs of it), then row form, then factor record.  The form comes
// before the record so that tasks that can share a wave are neighbours also
// where every problem has its own potential, i.e. every task its own record
// (150 subdomains of 40 to 127 cells, 20 potentials, 400 steps: 1.4 tasks in a wave
// of four slots by record, solve 3.17 ms and gradient 7.57; by form 2.66 and 5.59).
inline void sort_tasks(std::vector<Task>& list, const std::vector<int>& Pk, const std::vector<int>& rows) {
    std::stable_sort(list.begin(), list.end(), [&](const Task& x, const Task& y) {
        if (Pk[x.k] != Pk[y.k]) return Pk[x.k] > Pk[y.k];
        if (!rows.empty() && rows[x.k] != rows[y.k]) return rows[x.k] > rows[y.k];
        return x.f < y.f;
    });
}

// The workgroups of a task list that one kernel runs, whatever their widths.
struct RowsRun {
    int kind;             // RowsKind
    int pmax;             // widest of them (LDS size)
    int start, count;     // in the list's item table
};
struct RowsList {
    std::vector<int4> host;      // (first task, tasks, P, -)
    int4* dev = nullptr;
    std::vector<RowsRun> runs;
};
// A workgroup takes the tasks of one width that fit its waves (plain: one task);
// with the record in LDS, of one record.
inline void rows_items(const std::vector<int>& rows, const std::vector<Task>& list, bool plain, RowsList& out) {
    for (int kind = 0; kind < kRowsKinds; ++kind) {
        RowsRun run{kind, 0, (int)out.host.size(), 0};
        const RowsKind& rk = kRowsKind[kind];
        const int cap = plain ? 1 : rk.waves * (4 / rk.RW);
        for (size_t i = 0; i < list.size();) {
            const int key = rows[list[i].k], P = key % 32;
            if (key == 0 || key / 32 != rk.RW || (P >= kRowsLdsP) != rk.lds) { ++i; continue; }
            size_t j = i + 1;
            while (j < list.size() && (int)(j - i) < cap && rows[list[j].k] == key &&
                   (!rk.lds || list[j].f == list[i].f))
                ++j;
            out.host.push_back(make_int4((int)i, (int)(j - i), P, 0));
            run.pmax = std::max(run.pmax, P);
            i = j;
        }
        run.count = (int)out.host.size() - run.start;
        // widest first: the longest workgroups start first
        std::stable_sort(out.host.begin() + run.start, out.host.end(),
                         [](const int4& x, const int4& y) { return x.z > y.z; });
        if (run.count) out.runs.push_back(run);
    }
}

}  // namespace swr

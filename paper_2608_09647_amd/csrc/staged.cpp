// staged.cpp -- builds the staged column segments of a device matrix
// (kernels_staged.hip): row blocks, segment width, and per (block, segment,
// wave) the entries in row order with their turns in steps of 64.
#include <algorithm>
#include <atomic>
#include <climits>

#include "cgmi_host.h"

namespace cgmi {

namespace {

struct Entry {
    uint32_t idx;
    int32_t k;   // position in the CSR block
};

// The entries of a block as they go to the device.
struct BlockOut {
    HostVec<uint32_t> idx;
    HostVec<double> val;
    size_t n = 0;
    void push(uint32_t i, double v) {
        if (n == idx.size()) {
            idx.resize(n + n / 4 + 1024);
            val.resize(idx.size());
        }
        idx[n] = i;
        val[n++] = v;
    }
};

// Appends the entries of one (segment, wave) list to `out`, each with its
// turn: the entries its slot has in the same step of 64 before it.  A slot's
// ninth entry in a step starts a new step (the old one is padded with entries
// of the dummy slot).  seen[slot]: the step of the slot's last entry and its
// turn there; `step` numbers the steps of all lists that share `seen`.
void append_list(const Entry *in, size_t n, const double *val, uint32_t dummy, BlockOut &out,
                 std::vector<std::pair<uint32_t, uint32_t>> &seen, uint32_t &step) {
    const size_t first = out.n;
    ++step;
    for (size_t i = 0; i < n; ++i) {
        if (out.n > first && (out.n - first) % kWaveSize == 0) ++step;
        std::pair<uint32_t, uint32_t> &s = seen[staged_slot(in[i].idx)];
        uint32_t turn = s.first == step ? s.second + 1 : 0;
        if (turn == kStagedTurns) {
            while ((out.n - first) % kWaveSize) out.push(staged_word(0, 0, dummy), 0.0);
            ++step;
            turn = 0;
        }
        s = {step, turn};
        out.push(in[i].idx | turn << kStagedColBits, val[in[i].k]);
    }
}

}  // namespace

StagedShape staged_shape(int32_t m, int cus) {
    int32_t groups = 1;
    while (groups < 8 && (int64_t)m * groups * 2 <= (int64_t)cus * kStagedRows) groups *= 2;
    return {std::max<int32_t>((cus + groups - 1) / groups, (m + kStagedRows - 1) / kStagedRows), groups};
}

void staged_free(StagedMem &S) {
    (void)hipFree(const_cast<int32_t *>(S.dev.row0));
    (void)hipFree(const_cast<int32_t *>(S.dev.off));
    (void)hipFree(const_cast<uint32_t *>(S.dev.idx));
    (void)hipFree(const_cast<double *>(S.dev.val));
    (void)hipFree(const_cast<int32_t *>(S.dev.nslots));
    (void)hipFree(const_cast<uint32_t *>(S.dev.slots));
    (void)hipFree(S.dev.part);
    S.dev = StagedDev{};
    S.state = 0;
}

// state 1 on success; -1 where the matrix does not fit the layout or memory
// runs out (the products stay with the gathering kernels).
void staged_build(DevMatrix &M, int cus, StagedMem &S) {
    auto give_up = [&] {
        staged_free(S);
        S.state = -1;
    };
    give_up();
    const int32_t m = M.m;
    const int32_t max_seg = (int32_t)(16u * kStagedWaves * kWaveSize * kStagedChunks / sizeof(double));
    int32_t ncols = 0, longest = 0;
#pragma omp parallel for reduction(max : ncols, longest) schedule(static)
    for (int32_t i = 0; i < m; ++i) {
        longest = std::max(longest, M.h_rp[i + 1] - M.h_rp[i]);
        if (M.h_rp[i + 1] > M.h_rp[i]) ncols = std::max(ncols, M.h_ci[M.h_rp[i + 1] - 1] + 1);
    }
    if (longest > kHugeRow || ncols < 2 * max_seg) return;
    const StagedShape shape = staged_shape(m, cus);
    const int32_t nb = shape.nblocks, groups = shape.ngroups;
    const int32_t cap = std::min(kStagedMaxSlots - 1, kStagedRows * 5 / 4);
    try {
        // slots of a row: one per kStagedPerSlot entries a segment has of it on
        // average (of the shortest segments this can come to)
        const int32_t per_slot = kStagedPerSlot * ((ncols + max_seg - 1) / max_seg);
        auto len = [&](int32_t i) { return M.h_rp[i + 1] - M.h_rp[i]; };
        auto slots = [&](int32_t i) { return std::max(1, (len(i) + per_slot - 1) / per_slot); };
        // blocks of equal work (entries, and a little per row), at most cap slots
        std::vector<int32_t> row0((size_t)nb * kStagedWaves + 1, m), nslots((size_t)nb, 0);
        std::vector<uint32_t> slot_of((size_t)m);
        const double total = (double)M.nnz + 2.0 * m;
        int32_t max_slots = 1;
        bool several = false;
        {
            double done = 0.0;
            int32_t r = 0;
            for (int32_t b = 0; b < nb; ++b) {
                const int32_t first = r;
                const double before = done;
                int32_t u = 0;
                while (r < m && u + slots(r) <= cap && (b == nb - 1 || done < total * (b + 1) / nb)) {
                    const int32_t c = slots(r);
                    several |= c > 1;
                    slot_of[(size_t)r] = (uint32_t)u | (uint32_t)c << 16;
                    u += c;
                    done += len(r++) + 2.0;
                }
                nslots[(size_t)b] = u;
                max_slots = std::max(max_slots, u);
                const double work = done - before;
                double part = 0.0;
                int32_t q = first;
                for (int w = 0; w < kStagedWaves; ++w) {
                    row0[(size_t)b * kStagedWaves + w] = q;
                    while (q < r && (w == kStagedWaves - 1 || part < work * (w + 1) / kStagedWaves)) part += len(q++) + 2.0;
                }
            }
            if (r < m) return;   // the cap left rows over
        }
        const int32_t seg = staged_width(
            ncols, (int32_t)std::min<size_t>(max_seg, (kStagedLds - sizeof(double) * ((size_t)max_slots + 1)) /
                                                          (2 * sizeof(double))));
        if (!seg) return;
        const int32_t nseg = (ncols + seg - 1) / seg;
        if (nseg < groups) return;   // a group would have no segment, its first list none to begin at
        const int32_t lists = nseg * kStagedWaves;   // per block
        std::vector<int32_t> off((size_t)nb * lists + 1, 0);
        const int64_t room = M.nnz + M.nnz / 8;   // more padding than that does not pay
        if (room >= INT32_MAX - kStagedSlack) return;
        int32_t *d_row0 = nullptr, *d_off = nullptr, *d_nslots = nullptr;
        uint32_t *d_idx = nullptr, *d_slots = nullptr;
        double *d_val = nullptr;
        hipError_t e = staged_setup();
        if (e == hipSuccess) e = dmalloc(&d_row0, row0.size());
        S.dev.row0 = d_row0;
        if (e == hipSuccess) e = dmalloc(&d_nslots, nslots.size());
        S.dev.nslots = d_nslots;
        if (e == hipSuccess) e = dmalloc(&d_off, off.size());
        S.dev.off = d_off;
        if (e == hipSuccess) e = dmalloc(&d_idx, (size_t)room + kStagedSlack);
        S.dev.idx = d_idx;
        if (e == hipSuccess) e = dmalloc(&d_val, (size_t)room + kStagedSlack);
        S.dev.val = d_val;
        if (e == hipSuccess && several) e = dmalloc(&d_slots, slot_of.size());
        S.dev.slots = d_slots;
        if (e == hipSuccess) e = dmalloc(&S.dev.part, (size_t)groups * m);
        // a few blocks at a time: built by all threads, then uploaded
        const int32_t batch = 2 * omp_get_max_threads();
        std::vector<BlockOut> out((size_t)std::min(batch, nb));
        std::atomic<bool> ok{true};
        int64_t n = 0;
        for (int32_t b0 = 0; b0 < nb && e == hipSuccess; b0 += batch) {
            const int32_t b1 = std::min(nb, b0 + batch);
#pragma omp parallel
            {
                HostVec<Entry> raw;
                std::vector<int32_t> cnt;
                std::vector<std::pair<uint32_t, uint32_t>> seen;
#pragma omp for schedule(dynamic)
                for (int32_t b = b0; b < b1; ++b) {
                    try {
                        const int32_t *wr = &row0[(size_t)b * kStagedWaves];
                        const uint32_t dummy = (uint32_t)nslots[(size_t)b];
                        seen.assign((size_t)dummy + 1, {0, 0});
                        uint32_t step = 0;
                        cnt.assign((size_t)lists + 1, 0);
                        for (int w = 0; w < kStagedWaves; ++w)
                            for (int32_t k = M.h_rp[wr[w]]; k < M.h_rp[wr[w + 1]]; ++k)
                                ++cnt[(size_t)w * nseg + M.h_ci[k] / seg + 1];
                        for (int32_t l = 0; l < lists; ++l) cnt[(size_t)l + 1] += cnt[(size_t)l];
                        raw.resize((size_t)cnt[(size_t)lists]);
                        for (int w = 0; w < kStagedWaves; ++w)
                            for (int32_t i = wr[w]; i < wr[w + 1]; ++i) {
                                const uint32_t u = slot_of[(size_t)i] & 0xFFFFu, c = slot_of[(size_t)i] >> 16;
                                uint32_t t = 0;
                                for (int32_t k = M.h_rp[i]; k < M.h_rp[i + 1]; ++k) {
                                    const int32_t s = M.h_ci[k] / seg;
                                    raw[(size_t)cnt[(size_t)w * nseg + s]++] =
                                        Entry{staged_word((uint32_t)(M.h_ci[k] - s * seg), 0, u + t), k};
                                    if (++t == c) t = 0;
                                }
                            }
                        BlockOut &o = out[(size_t)(b - b0)];
                        o.n = 0;
                        for (int32_t l = 0; l < lists; ++l) {   // cnt[l] is the end of list l by now
                            const int32_t beg = l ? cnt[(size_t)l - 1] : 0;
                            append_list(raw.data() + beg, (size_t)(cnt[(size_t)l] - beg), M.h_val.data(), dummy, o,
                                           seen, step);
                            off[(size_t)b * lists + l + 1] = (int32_t)o.n;
                        }
                    } catch (...) {
                        ok = false;
                    }
                }
            }
            if (!ok.load()) return give_up();
            for (int32_t b = b0; b < b1 && e == hipSuccess; ++b) {
                const BlockOut &o = out[(size_t)(b - b0)];
                if (n + (int64_t)o.n > room) return give_up();
                for (int32_t l = 0; l < lists; ++l) off[(size_t)b * lists + l + 1] += (int32_t)n;
                if (o.n) e = hipMemcpy(d_idx + n, o.idx.data(), sizeof(uint32_t) * o.n, hipMemcpyHostToDevice);
                if (o.n && e == hipSuccess)
                    e = hipMemcpy(d_val + n, o.val.data(), sizeof(double) * o.n, hipMemcpyHostToDevice);
                n += (int64_t)o.n;
            }
        }
        if (e == hipSuccess) e = hipMemcpy(d_row0, row0.data(), sizeof(int32_t) * row0.size(), hipMemcpyHostToDevice);
        if (e == hipSuccess)
            e = hipMemcpy(d_nslots, nslots.data(), sizeof(int32_t) * nslots.size(), hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(d_off, off.data(), sizeof(int32_t) * off.size(), hipMemcpyHostToDevice);
        if (e == hipSuccess && several)
            e = hipMemcpy(d_slots, slot_of.data(), sizeof(uint32_t) * slot_of.size(), hipMemcpyHostToDevice);
        // entry 0 of the padding: column 0, turn 0, slot 0, never on
        if (e == hipSuccess) e = hipMemset(d_idx + n, 0, sizeof(uint32_t) * kStagedSlack);
        if (e == hipSuccess) e = hipMemset(d_val + n, 0, sizeof(double) * kStagedSlack);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return give_up();
        }
        S.dev.m = m;
        S.dev.nblocks = nb;
        S.dev.ngroups = groups;
        S.dev.nseg = nseg;
        S.dev.seg_cols = seg;
        S.dev.max_slots = max_slots;
        S.dev.ncols = ncols;
        S.dev.ahead = (int32_t)(n / ((int64_t)nb * lists) / kWaveSize) + 1;
        S.state = 1;
    } catch (...) {
        give_up();
    }
}

}  // namespace cgmi

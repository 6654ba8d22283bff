// Host-side plan of the LDS-halo SpMM (k_spmm_halo): consecutive CSR rows, each
// with at most emax entries, are grouped greedily into blocks of at most rmax
// rows whose halo (the distinct columns of the rows together with the rows
// themselves, kept sorted) numbers at most hmax entries.  The block's rows
// then sit at consecutive halo slots from rbase[b]; lcol[e] is the slot of
// entry e's column in its block's halo.  Plain C++ (no HIP), so the host
// tests compile it with g++.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

namespace ofks {

struct HaloPlan {
    std::vector<int64_t> row0{0};   // block b owns rows [row0[b], row0[b+1])
    std::vector<int64_t> hoff{0};   // block b's halo is halo[hoff[b] .. hoff[b+1])
    std::vector<int32_t> halo;      // ascending within a block
    std::vector<uint16_t> lcol;     // per CSR entry
    std::vector<int32_t> rbase;     // halo slot of block b's first row
    int64_t nb() const { return (int64_t)row0.size() - 1; }
};

enum { HALO_OK = 0, HALO_TOO_WIDE = 1, HALO_BAD_ROWPTR = -1, HALO_BAD_COLUMN = -2, HALO_BAD_PLAN = -3 };

// Build the plan.  HALO_TOO_WIDE: some row has more than emax entries or
// alone a halo of more than hmax (no plan); HALO_BAD_*: the CSR arrays
// are malformed (*where = row or entry).  hmax <= 65536 so that a slot fits in
// 16 bits.
inline int halo_plan_build(int64_t n, const int64_t *rp, const int32_t *col, int hmax, int rmax, int emax,
                           HaloPlan &P, int64_t *where) {
    P = HaloPlan();
    if (n <= 0 || rp[0] != 0) { *where = 0; return HALO_BAD_ROWPTR; }
    const int64_t nnz = rp[n];
    if (hmax < 1 || hmax > 65536 || rmax < 1) { *where = 0; return HALO_BAD_PLAN; }
    std::vector<int64_t> stamp(n, -1);   // b: in block b's halo
    std::vector<int32_t> slot(n, 0);
    std::vector<int32_t> cur, words;
    std::vector<uint64_t> bits((size_t)(n + 63) / 64, 0);
    P.lcol.assign((size_t)std::max<int64_t>(nnz, 0), 0);
    P.halo.reserve((size_t)(3.5 * n) + 64);
    int64_t b = 0, start = 0;
    auto close = [&](int64_t end) {
        // ascending order by way of a bitmap: only its few touched words are sorted
        words.clear();
        for (const int32_t c : cur) {
            if (!bits[c >> 6]) words.push_back(c >> 6);
            bits[c >> 6] |= uint64_t(1) << (c & 63);
        }
        std::sort(words.begin(), words.end());
        int32_t k = 0;
        for (const int32_t w : words) {
            for (uint64_t m = bits[w]; m; m &= m - 1, ++k) {
                cur[k] = 64 * w + __builtin_ctzll(m);
                slot[cur[k]] = k;
            }
            bits[w] = 0;
        }
        for (int64_t e = rp[start]; e < rp[end]; ++e) P.lcol[e] = (uint16_t)slot[col[e]];
        P.rbase.push_back(slot[start]);
        P.halo.insert(P.halo.end(), cur.begin(), cur.end());
        P.row0.push_back(end);
        P.hoff.push_back((int64_t)P.halo.size());
        cur.clear();
        ++b;
        start = end;
    };
    for (int64_t r = 0; r < n; ++r) {
        if (rp[r + 1] < rp[r] || rp[r + 1] > nnz) { *where = r; return HALO_BAD_ROWPTR; }
        if (rp[r + 1] - rp[r] > emax) { *where = r; P = HaloPlan(); return HALO_TOO_WIDE; }
        for (int pass = 0;; ++pass) {
            if (r - start < rmax) {
                const size_t mark = cur.size();
                for (int64_t e = rp[r]; e <= rp[r + 1]; ++e) {   // the entries, then the row itself
                    const int64_t cc = e < rp[r + 1] ? col[e] : r;
                    if (cc < 0 || cc >= n) { *where = e; return HALO_BAD_COLUMN; }
                    if (stamp[cc] != b) {
                        stamp[cc] = b;
                        cur.push_back((int32_t)cc);
                    }
                }
                if ((int64_t)cur.size() <= hmax) break;
                for (size_t k = mark; k < cur.size(); ++k) stamp[cur[k]] = -1;   // the row does not fit
                cur.resize(mark);
            }
            if (pass == 1 || r == start) { *where = r; P = HaloPlan(); return HALO_TOO_WIDE; }
            close(r);   // the row opens the next block
        }
    }
    close(n);
    return HALO_OK;
}

// Independent check of a plan against the CSR arrays: every row covered once,
// block and row sizes within bounds, every slot in range and mapping back to
// its column, the block's rows at slots rbase[b] + (r - row0[b]).
inline int halo_plan_check(int64_t n, const int64_t *rp, const int32_t *col, int hmax, int rmax, int emax,
                           const HaloPlan &P, int64_t *where) {
    const int64_t nb = P.nb();
    if (nb < 1 || P.row0[0] != 0 || P.row0[nb] != n || (int64_t)P.hoff.size() != nb + 1 || P.hoff[0] != 0 ||
        P.hoff[nb] != (int64_t)P.halo.size() || (int64_t)P.lcol.size() != rp[n] || (int64_t)P.rbase.size() != nb) {
        *where = -1;
        return HALO_BAD_PLAN;
    }
    for (int64_t k = 0; k < nb; ++k) {
        const int64_t hn = P.hoff[k + 1] - P.hoff[k];
        if (P.row0[k + 1] <= P.row0[k] || P.row0[k + 1] - P.row0[k] > rmax || hn < P.row0[k + 1] - P.row0[k] ||
            hn > hmax || P.rbase[k] < 0 || P.rbase[k] + (P.row0[k + 1] - P.row0[k]) > hn) {
            *where = k;
            return HALO_BAD_PLAN;
        }
        for (int64_t r = P.row0[k]; r < P.row0[k + 1]; ++r)
            if (P.halo[P.hoff[k] + P.rbase[k] + (r - P.row0[k])] != r) {
                *where = r;
                return HALO_BAD_PLAN;
            }
        for (int64_t r = P.row0[k]; r < P.row0[k + 1]; ++r)
            if (rp[r + 1] - rp[r] > emax) {
                *where = r;
                return HALO_BAD_PLAN;
            }
        for (int64_t e = rp[P.row0[k]]; e < rp[P.row0[k + 1]]; ++e)
            if (P.lcol[e] >= hn || P.halo[P.hoff[k] + P.lcol[e]] != col[e]) {
                *where = e;
                return HALO_BAD_PLAN;
            }
    }
    return HALO_OK;
}

// Whether the LDS-halo product of a block of p columns of `elem` bytes beats the
// row-gather product, by the plan's halo rows per matrix row (15-entry rows:
// Z-order numbering 3.1, Delaunay meshes so numbered 3.7, lexicographic 7.2,
// Z-order shuffled within windows of 64, 128, 256 and 1024 rows 3.4, 7.3, 10.4
// and 13.2, random 14.3).  Each halo row is staged whatever its use, while the
// gathered rows come from caches.  Measured, gather against halo, us, n = 2.05e5:
//   up to 5: FP64 from p = 4 on (Z-order, dual product: p = 4 66 and 47, 11 73 and
//     57, 32 74 and 53, 128 274 and 164), FP32 from p = 33 on (33 161 and 61, 64 63
//     and 51, 128 151 and 77), below which a row of X fills a small part of the
//     staged 256-byte slots
//   up to 9: FP64 from p = 24 on (lexicographic, dual and shifted product: p = 8 51
//     and 64, 58 and 74; 16 51 and 63, 60 and 72; 24 74 and 64, 86 and 73; 64 156 and
//     111, 147 and 114); FP32 past p = 128 and at odd p, where the gather takes
//     single values (33 162 and 94, 175 and 105; 64 64 and 68, 75 and 85; 128 138 and
//     118, 115 and 137; 160 187 and 154, 224 and 180)
//   above: FP64 from p = 64 on (random: p = 11 98 and 156, 110 and 173; 48 200 and
//     234, 198 and 238; 64 265 and 253, 258 and 254; 128 511 and 492, 513 and 462);
//     FP32 never (96 198 and 232, 199 and 272; 160 319 and 368, 327 and 412)
inline bool halo_product_pays(int64_t n, int64_t halo_rows, int p, int elem) {
    if (halo_rows <= 5 * n) return elem == 8 ? p >= 4 : p >= 33;
    if (halo_rows <= 9 * n) return elem == 8 ? p >= 24 : p > 128 || (p >= 33 && p % 2);
    return elem == 8 && p >= 64;
}

// Whether the one-kernel Hartree CG iteration, which reads a row's state once per
// halo that it lies in, beats product, update and direction kernels.  Ten
// iterations, us, here against those three: Z-order n = 1.0e5 108 and 191, 5.1e5
// 293 and 432, 2.0e6 1336 and 1686; lexicographic 1.0e5 142 and 194, 2.1e5 (1.5e6
// halo rows) 227 and 262, 5.1e5 (3.7e6) 467 and 429, 2.0e6 2108 and 1692; random
// 4.3e4 (0.6e6) 140 and 159, 1.0e5 (1.5e6) 265 and 221, 1.0e6 2612 and 1841.
inline bool halo_cg_pays(int64_t n, int64_t halo_rows) {
    return halo_rows <= 4 * n || halo_rows <= 1000000 || (halo_rows <= 8 * n && halo_rows <= 2000000);
}

}  // namespace ofks

// Host-only logic of the library (layouts, chunk plan, metadata builder, validation) run on exact-size buffers
// under AddressSanitizer / UBSan.  Built and run by tests/test_host_asan.py; no GPU involved.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <cstdint>
#include <cstdlib>
#include <vector>

#include "hr_attn_rows.h"
#include "hr_gemm_tiles.h"
#include "hr_internal.h"

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); return 1; } } while (0)

int main() {
    // chunk plan of mixed lengths, metadata written into a buffer of exactly the computed size
    std::vector<int32_t> lens = {270, 4, 64, 65, 128, 2112, 1};
    for (int chunk : {32, 64}) {
        hr::ChunkPlan cp = hr::make_chunk_plan((int64_t)lens.size(), lens.data(), chunk);
        hr::MetaLayout ml = hr::make_meta_layout(cp.n_chunks, cp.T, cp.pt_stride, (int64_t)lens.size(), 10);
        std::vector<int32_t> meta(ml.total, -7), toks(cp.T, 1);
        hr::fill_meta(meta.data(), ml, cp.n_chunks, cp.prefix_lens.data(), cp.new_lens.data(), toks.data(), cp.page_table.data(),
                      cp.pt_stride, cp.out_row.data(), (int64_t)lens.size());
        int64_t total = 0;
        for (int32_t l : lens) total += l;
        CHECK(cp.T == total);
        CHECK(meta[ml.cu + cp.n_chunks] == total);
        // every chunk starts on a 32-slot boundary and a sequence's pages are contiguous
        int64_t ci = 0;
        for (size_t s = 0; s < lens.size(); ++s) {
            for (int64_t off = 0; off < lens[s]; off += chunk, ++ci) {
                CHECK(meta[ml.new_cu + ci] % 32 == 0);
                CHECK(meta[ml.new_cu + ci] == cp.first_page[s] * 16 + off);
                CHECK(meta[ml.prefix_len + ci] == off);
                for (int64_t pg = 0; pg < off / 16; ++pg) CHECK(meta[ml.page_table + ci * cp.pt_stride + pg] == cp.first_page[s] + pg);
            }
            CHECK(meta[ml.out_row + s] == meta[ml.cu + ci] - 1);
        }
    }
    // scoring layout: positions continue after the document, slots are 32-aligned per pair
    std::vector<int32_t> dl = {100, 0, 17}, ql = {5, 1, 33}, pt(3 * 7, 3), tk(39, 2);
    hr::MetaLayout m2 = hr::make_meta_layout(3, 39, 7);
    std::vector<int32_t> meta2(m2.total);
    hr::fill_meta(meta2.data(), m2, 3, dl.data(), ql.data(), tk.data(), pt.data(), 7);
    CHECK(meta2[m2.tok_pos + 0] == 100 && meta2[m2.tok_pos + 4] == 104 && meta2[m2.tok_pos + 5] == 0 && meta2[m2.tok_pos + 6] == 17);
    CHECK(meta2[m2.new_cu + 0] == 0 && meta2[m2.new_cu + 1] == 32 && meta2[m2.new_cu + 2] == 64 && meta2[m2.new_cu + 3] == 128);
    CHECK(meta2[m2.out_row + 0] == 4 && meta2[m2.out_row + 1] == 5 && meta2[m2.out_row + 2] == 38);
    // group plan: pairs with identical page-table rows and lengths share a group up to the block capacity; every
    // block and every 32-key sub-tile of every pair appears exactly once; groups come heaviest first
    {
        const int g = 7, cap = 16, stride = 4;
        // docs: A = pages {3, 9}, len 30; B = pages {5}, len 16; pair 6 has A's first page but another second page
        std::vector<int32_t> gd = {30, 16, 30, 0, 30, 16, 30, 0, 30}, gq = {40, 8, 33, 5, 64, 1, 9, 5, 20};
        std::vector<int32_t> gpt = {3, 9, -1, -1, 5, -1, -1, -1, 3, 9, -1, -1, -1, -1, -1, -1, 3, 9, -1, -1, 5, -1, -1, -1,
                                    3, 8, -1, -1, -1, -1, -1, -1, 3, 9, -1, -1};
        const int64_t n = (int64_t)gd.size();
        int64_t Tq = 0;
        for (int32_t v : gq) Tq += v;
        hr::GroupPlan gp = hr::make_group_plan(n, gd.data(), gq.data(), gpt.data(), stride, g, cap);
        CHECK(gp.ints() <= hr::group_plan_ints_bound(n, Tq, g));
        std::vector<int32_t> flat(gp.ints(), -7);
        hr::store_group_plan(gp, flat.data());
        CHECK(flat[0] == gp.p0[0] && flat.back() == gp.sub_key0.back());
        CHECK(gp.shared && gp.max_blocks <= cap);
        CHECK((int)gp.blk_cu.size() == gp.n_groups + 1 && (int)gp.sub_cu.size() == gp.n_groups + 1);
        std::vector<int> blocks_seen(n, 0), subs_seen(n, 0), group_of(n, -1);
        int64_t prev_cost = INT64_MAX;
        std::vector<int64_t> new_page(n);
        int64_t slot = 0;
        for (int64_t p = 0; p < n; ++p) { new_page[p] = slot / 16; slot += (gq[p] + 31) / 32 * 32; }
        for (int gi = 0; gi < gp.n_groups; ++gi) {
            const int32_t lead = gp.p0[gi];
            const int nb = gp.blk_cu[gi + 1] - gp.blk_cu[gi];
            CHECK(nb >= 1 && nb <= cap);
            const int64_t cost = ((int64_t)gd[lead] + 64) * nb;
            CHECK(cost <= prev_cost);
            prev_cost = cost;
            for (int b = gp.blk_cu[gi]; b < gp.blk_cu[gi + 1]; ++b) {
                const int32_t p = gp.blk_seq[b];
                CHECK(p >= 0 && p < n && gd[p] == gd[lead]);
                for (int pg = 0; pg < (gd[p] + 15) / 16; ++pg) CHECK(gpt[p * stride + pg] == gpt[lead * stride + pg]);
                CHECK(group_of[p] == -1 || group_of[p] == gi);
                group_of[p] = gi;
                CHECK(gp.blk_row0[b] == 32 * blocks_seen[p]);              // a pair's blocks in order, back to back
                CHECK(b == gp.blk_cu[gi] || gp.blk_seq[b - 1] == p || blocks_seen[p] == 0);
                ++blocks_seen[p];
            }
            for (int s = gp.sub_cu[gi]; s < gp.sub_cu[gi + 1]; ++s) {
                const int32_t p = gp.sub_seq[s];
                CHECK(group_of[p] == gi);
                CHECK(gp.sub_key0[s] == 32 * subs_seen[p] && gp.sub_page[s] == new_page[p] + 2 * subs_seen[p]);
                ++subs_seen[p];
            }
        }
        for (int64_t p = 0; p < n; ++p) {
            CHECK(blocks_seen[p] == (gq[p] * g + 31) / 32 && subs_seen[p] == (gq[p] + 31) / 32);
            if (gd[p] == 0) CHECK(gp.blk_cu[group_of[p] + 1] - gp.blk_cu[group_of[p]] == blocks_seen[p]);   // no document: alone
        }
        // A is shared by pairs 0, 2, 4, 8 (9 + 8 + 14 + 5 blocks): at least two groups; pair 6 is not with them
        CHECK(group_of[6] != group_of[0] && group_of[6] != group_of[2] && group_of[6] != group_of[4] && group_of[6] != group_of[8]);
        CHECK(group_of[1] == group_of[5]);
        CHECK(group_of[3] != group_of[7]);
        // nothing shared: every pair alone
        std::vector<int32_t> upt = {1, 2, 3};
        std::vector<int32_t> ud = {16, 16, 16}, uq = {4, 4, 4};
        hr::GroupPlan up = hr::make_group_plan(3, ud.data(), uq.data(), upt.data(), 1, g, cap);
        CHECK(!up.shared && up.n_groups == 3 && up.max_blocks == 1);
        CHECK(!up.uneven && gp.uneven);
        // scarce work items: sequences are cut into pieces of at most 4 blocks; every (sequence, block) exactly once, and
        // every group lists the own keys of each of its sequences exactly once
        hr::GroupPlan cp4 = hr::make_group_plan(n, gd.data(), gq.data(), gpt.data(), stride, g, 4, true);
        CHECK(cp4.cut && cp4.max_blocks <= 4 && cp4.ints() <= hr::group_plan_ints_bound(n, Tq, g));
        std::vector<std::vector<char>> seen(n);
        for (int64_t p = 0; p < n; ++p) seen[p].assign((gq[p] * g + 31) / 32, 0);
        for (int gi = 0; gi < cp4.n_groups; ++gi) {
            std::vector<int> subs_in_group(n, 0), blocks_in_group(n, 0);
            for (int b = cp4.blk_cu[gi]; b < cp4.blk_cu[gi + 1]; ++b) {
                const int32_t p = cp4.blk_seq[b];
                CHECK(cp4.blk_row0[b] % 32 == 0 && cp4.blk_row0[b] / 32 < (int)seen[p].size() && !seen[p][cp4.blk_row0[b] / 32]);
                seen[p][cp4.blk_row0[b] / 32] = 1;
                CHECK(gd[p] == gd[cp4.p0[gi]]);
                ++blocks_in_group[p];
            }
            for (int sidx = cp4.sub_cu[gi]; sidx < cp4.sub_cu[gi + 1]; ++sidx) {
                const int32_t p = cp4.sub_seq[sidx];
                CHECK(cp4.sub_key0[sidx] == 32 * subs_in_group[p] && cp4.sub_page[sidx] == new_page[p] + 2 * subs_in_group[p]);
                ++subs_in_group[p];
            }
            for (int64_t p = 0; p < n; ++p) CHECK(subs_in_group[p] == (blocks_in_group[p] ? (gq[p] + 31) / 32 : 0));
        }
        for (int64_t p = 0; p < n; ++p)
            for (char c : seen[p]) CHECK(c == 1);
        // many sequences of up to 16 blocks cut into pieces of at most 8 (128-wide heads): fits the room reserved for a plan
        {
            const int64_t nn = 300;
            const int g8 = 8;
            std::vector<int32_t> md(nn), mq(nn), mpt(nn);
            int64_t Tm = 0;
            for (int64_t p = 0; p < nn; ++p) {
                md[p] = 16;
                mq[p] = 1 + (int32_t)((p * 37) % 64);
                mpt[p] = (int32_t)(p % 7);                   // a few shared first pages (same length: shared documents)
                Tm += mq[p];
            }
            hr::GroupPlan cp8 = hr::make_group_plan(nn, md.data(), mq.data(), mpt.data(), 1, g8, 8, true);
            CHECK(cp8.cut && cp8.max_blocks <= 8 && cp8.ints() <= hr::group_plan_ints_bound(nn, Tm, g8));
            std::vector<int> blocks(nn, 0);
            for (size_t b = 0; b < cp8.blk_seq.size(); ++b) ++blocks[cp8.blk_seq[b]];
            for (int64_t p = 0; p < nn; ++p) CHECK(blocks[p] == (mq[p] * g8 + 31) / 32);
        }
        std::vector<int32_t> rd = {16, 48, 32};                   // nothing shared, lengths differ: heaviest first
        hr::GroupPlan rp = hr::make_group_plan(3, rd.data(), uq.data(), upt.data(), 1, g, cap);
        CHECK(!rp.shared && rp.uneven && rp.p0[0] == 1 && rp.p0[1] == 2 && rp.p0[2] == 0);
    }
    // a call cut in two halves: the two carvings fit the whole call's workspace plus the 1 MB the size query adds
    {
        hr_model_cfg mcs[2] = {{24, 896, 14, 2, 64, 4864, 1000, 1, 2, HR_BF16, 1e6f, 1e-6f}, {32, 4096, 32, 8, 128, 14336, 1000, 1, 2, HR_BF16, 5e5f, 1e-5f}};
        unsigned rs = 12345u;
        auto rnd = [&](unsigned n) { rs = rs * 1664525u + 1013904223u; return (rs >> 8) % n; };
        for (int it = 0; it < 400; ++it) {
            const hr_model_cfg& mc2 = mcs[it & 1];
            const int g2 = mc2.n_q_heads / mc2.n_kv_heads;
            const int64_t n = 2 + rnd(3000), T = n + rnd(40000), stride = 1 + rnd(130);
            const int64_t na = 1 + rnd((unsigned)(n - 1)), Ta = na + rnd((unsigned)(T - n + 1));       // Ta >= na, Tb >= nb
            const int64_t nb = n - na, Tb = T - Ta;
            if (Tb < nb) continue;
            const size_t whole = hr::make_workspace(mc2, n, T, stride, false, -1, 0, (int64_t)hr::group_plan_ints_bound(n, T, g2)).total;
            const size_t a_part = hr::make_workspace(mc2, na, Ta, stride, false, -1, 0, (int64_t)hr::group_plan_ints_bound(na, Ta, g2)).total;
            const size_t b_part = hr::make_workspace(mc2, nb, Tb, stride, false, -1, 0, (int64_t)hr::group_plan_ints_bound(nb, Tb, g2)).total;
            CHECK(a_part + b_part <= whole + (1 << 20));
        }
    }
    // pool bookkeeping and validation paths
    hr_pool_cfg pc{2, 2, 64, 16, 8, HR_BF16};
    hr_pool* pool = nullptr;
    CHECK(hr_kv_pool_create(&pc, (void*)0x1000, hr_kv_pool_bytes(&pc), &pool) == HR_OK);
    int32_t ids[3] = {1, 5, 1};
    CHECK(hr::pool_check_write(pool, 40, ids) == HR_ERR_PAGE_DUP);
    ids[2] = 7;
    CHECK(hr::pool_check_write(pool, 40, ids) == HR_OK);
    CHECK(hr::pool_check_read(pool, 40, ids) == HR_ERR_TABLE_SHORT);
    hr::pool_mark(pool, ids, 3, hr::PAGE_USED);
    CHECK(hr_kv_pool_free_pages(pool) == 5);
    CHECK(hr::pool_check_read(pool, 40, ids) == HR_OK);
    CHECK(hr::pool_check_read(pool, 0, ids) == HR_ERR_LEN_RANGE);
    hr_model_cfg mc{2, 128, 4, 2, 64, 256, 100, 1, 2, HR_BF16, 10000.f, 1e-6f};
    int32_t table[2 * 3] = {1, 5, 7, 1, 5, -1};
    int32_t dls[2] = {40, 32}, qls[2] = {3, 2}, qt[5] = {1, 2, 3, 4, 99};
    int64_t T = 0;
    CHECK(hr::score_check_args(mc, pool, 2, table, 3, dls, qt, qls, 1 << 20, &T) == HR_OK && T == 5);
    qt[4] = 100;
    CHECK(hr::score_check_args(mc, pool, 2, table, 3, dls, qt, qls, 1 << 20, &T) == HR_ERR_TOKEN_RANGE);
    dls[1] = 48;
    CHECK(hr::score_check_args(mc, pool, 2, table, 3, dls, qt, qls, 1 << 20, &T) == HR_ERR_TABLE_SHORT);
    hr_kv_pool_destroy(pool);

    // the measure by which a call is cut in two halves follows the launches: in (0, 1], 1 where they leave no slot empty
    {
        std::srand(7);
        for (int it = 0; it < 2000; ++it) {
            const int64_t M = 1 + std::rand() % 120000;
            const int N = 64 * (1 + std::rand() % 480), ko = 64 * (1 + std::rand() % 80), kd = 64 * (1 + std::rand() % 230);
            const double fill = hr::gemm_resid_fill(M, N, ko, kd, 8 * (1 + std::rand() % 40));
            CHECK(fill > 0.0 && fill <= 1.0);
        }
        CHECK(hr::gemm_resid_fill(20480, 896, 896, 4864, 256) == 1.0);          // 320 x 256: 256 tiles, one round
        // 8B shape, 12800 tokens: three rounds of 256 x 256 and one of 64 x 128 for the last 512 rows, no slot empty
        const hr::GemmLaunch d8 = hr::choose_gemm_launch(hr::GEMM_RESID, 12800, 4096, 14336, 256);
        CHECK(d8.n == 2 && d8.part[0].rows == 12288 && d8.part[1].rows == 512);
        CHECK(hr::gemm_resid_fill(12800, 4096, 4096, 14336, 256) == 1.0);
        // 0.5B shape, 10240 tokens: O as 560 tiles of 128 x 128 in two rounds of 512, down as 160 tiles of 256 x 256 in one
        const double f = hr::gemm_resid_fill(10240, 896, 896, 4864, 256);
        CHECK(f > 0.59 && f < 0.62);
    }
    {   // GEMM launches: the parts cover the rows, in order, with shapes the epilogue has; a cut leaves whole rounds in front
        std::srand(11);
        const hr::GemmKind kinds[] = {hr::GEMM_QKV64, hr::GEMM_QKV128, hr::GEMM_RESID, hr::GEMM_SWIGLU};
        int cuts[4] = {0, 0, 0, 0};
        for (int it = 0; it < 8000; ++it) {
            const hr::GemmKind kind = kinds[it % 4];
            const int64_t M = it % 8 < 4 ? 1 + std::rand() % 3000 : 1 + std::rand() % 120000;
            const int N = 64 * (1 + std::rand() % 480), K = 64 * (1 + std::rand() % 230), cus = 8 * (1 + std::rand() % 40);
            const hr::GemmLaunch g = hr::choose_gemm_launch(kind, M, N, K, cus, it % 16 >= 12);
            CHECK(g.n == 1 || g.n == 2);
            int64_t rows = 0;
            for (int i = 0; i < g.n; ++i) {
                const hr::GemmPart& p = g.part[i];
                const hr::GemmTile t = p.tile;
                CHECK(p.rows > 0 && p.bm >= 32 && p.bm % 32 == 0 && p.bn >= 32 && p.bn % 32 == 0);
                if (t == hr::GT_RING32_64 || t == hr::GT_RING32_128) {      // one tile per CU
                    CHECK(p.bm == 32 && p.bn == (t == hr::GT_RING32_64 ? 64 : 128));
                    CHECK((p.rows + 31) / 32 * ((N + p.bn - 1) / p.bn) <= cus);
                }
                rows += g.part[i].rows;
                switch (kind) {
                    case hr::GEMM_QKV64: CHECK(t == hr::GT_BIG || t == hr::GT_SMALL || t == hr::GT_RING128 || t == hr::GT_RING64 || t == hr::GT_RING32_64); break;
                    case hr::GEMM_QKV128: CHECK(t == hr::GT_BIG || t == hr::GT_RING128 || t == hr::GT_RING64_128 || t == hr::GT_RING32_128); break;
                    case hr::GEMM_RESID:
                        CHECK(t == hr::GT_BIG || t == hr::GT_TALL || t == hr::GT_SMALL || t == hr::GT_RING128 || t == hr::GT_RING64_128 ||
                              ((t == hr::GT_RING160_64 || t == hr::GT_RING96_64) && K >= 512) || t == hr::GT_RING64 || t == hr::GT_RING32);
                        break;
                    case hr::GEMM_SWIGLU:
                        CHECK(t == hr::GT_BIG || (t == hr::GT_TALL && K >= 2048) || t == hr::GT_SMALL || t == hr::GT_RING128_256 ||
                              t == hr::GT_RING128 || t == hr::GT_RING64_128);
                        break;
                }
            }
            CHECK(rows == M);
            if (g.n == 2) {
                ++cuts[it % 4];
                const hr::GemmTile t = g.part[0].tile;
                CHECK(t == hr::GT_BIG || t == hr::GT_TALL);
                const int64_t bm = t == hr::GT_TALL ? 320 : 256, tn = (N + 255) / 256;
                CHECK(g.part[0].rows % bm == 0);
                const int64_t tiles = g.part[0].rows / bm * tn, part = tiles % cus;
                CHECK(tiles > cus - tn && (part == 0 || part > cus - tn));       // the cut lies at the last whole row of tiles
            }
        }
        for (int c : cuts) CHECK(c > 0);
        // the launches that the GPU tests of cut projections rely on
        CHECK(hr::choose_gemm_launch(hr::GEMM_SWIGLU, 1980, 2 * 4864, 896, 256).n == 2);
        CHECK(hr::choose_gemm_launch(hr::GEMM_QKV64, 6600, 2560, 512, 256).n == 2);
        CHECK(hr::choose_gemm_launch(hr::GEMM_QKV128, 12000, 1536, 256, 256).n == 2);
        // halves of a call, 0.5B shape: tiles that share a CU, whatever a launch with the chip to itself would take
        for (int64_t M = 4704; M <= 5760; M += 4) {
            const hr::GemmLaunch alone = hr::choose_gemm_launch(hr::GEMM_RESID, M, 896, 4864, 256), half = hr::choose_gemm_launch(hr::GEMM_RESID, M, 896, 4864, 256, true);
            CHECK(alone.n == 1 && alone.part[0].tile == hr::GT_RING160_64 && half.n == 1 && half.part[0].tile == hr::GT_SMALL);
        }
        const hr::GemmLaunch gu = hr::choose_gemm_launch(hr::GEMM_SWIGLU, 5720, 2 * 4864, 896, 256, true);
        CHECK(gu.n == 2 && gu.part[0].tile == hr::GT_BIG && gu.part[1].tile == hr::GT_SMALL);
        // ... and those of single tile shapes
        struct Pin { hr::GemmKind kind; int64_t M; int N, K; hr::GemmTile tile; };
        const Pin pins[] = {
            {hr::GEMM_RESID, 1980, 896, 4864, hr::GT_RING64_128},  {hr::GEMM_RESID, 205, 256, 4864, hr::GT_RING32},
            {hr::GEMM_RESID, 350, 320, 4160, hr::GT_RING32},
            // tiles for few rows
            {hr::GEMM_RESID, 1295, 896, 896, hr::GT_RING96_64},    {hr::GEMM_RESID, 1295, 896, 2112, hr::GT_RING96_64},
            {hr::GEMM_RESID, 2460, 896, 896, hr::GT_RING160_64},   {hr::GEMM_RESID, 2460, 896, 576, hr::GT_RING160_64},
            {hr::GEMM_QKV64, 165, 512, 256, hr::GT_RING32_64},     {hr::GEMM_QKV128, 175, 1536, 2048, hr::GT_RING32_128},
            // blocked weights
            {hr::GEMM_RESID, 175, 2048, 2048, hr::GT_RING64},      {hr::GEMM_RESID, 37, 2048, 2112, hr::GT_RING32},
            {hr::GEMM_RESID, 1295, 2048, 2112, hr::GT_RING128},
            // W read ahead of the ring
            {hr::GEMM_RESID, 1295, 896, 17600, hr::GT_RING96_64},  {hr::GEMM_RESID, 2460, 896, 17600, hr::GT_RING160_64},
            {hr::GEMM_RESID, 4290, 896, 4864, hr::GT_RING128},     {hr::GEMM_RESID, 330, 2048, 8192, hr::GT_RING64},
            {hr::GEMM_RESID, 700, 2048, 8192, hr::GT_RING96_64},   {hr::GEMM_RESID, 1260, 2048, 8192, hr::GT_RING160_64},
            {hr::GEMM_RESID, 1295, 2048, 8192, hr::GT_RING128},    {hr::GEMM_QKV128, 330, 2560, 2048, hr::GT_RING32_128},
            {hr::GEMM_QKV128, 700, 2560, 2048, hr::GT_RING64_128}, {hr::GEMM_QKV128, 1260, 2560, 2048, hr::GT_RING128},
            {hr::GEMM_SWIGLU, 4290, 640, 2048, hr::GT_RING128},    {hr::GEMM_QKV128, 4290, 1536, 2048, hr::GT_RING128}};
        for (const Pin& p : pins) {
            const hr::GemmLaunch g = hr::choose_gemm_launch(p.kind, p.M, p.N, p.K, 256);
            CHECK(g.n == 1 && g.part[0].tile == p.tile);
        }
    }
    {   // 256-row residual tiles of 224 columns: the calls of the GPU test, and where 256-wide ones stay (fewer columns, blocked weights)
        struct Narrow { int64_t M; int N, K, bn; };
        for (const Narrow& c : {Narrow{6600, 1344, 1792, 224}, Narrow{9900, 832, 2432, 224}, Narrow{16384, 1024, 4864, 256}, Narrow{12288, 4096, 14336, 256}}) {
            const hr::GemmLaunch g = hr::choose_gemm_launch(hr::GEMM_RESID, c.M, c.N, c.K, 256);
            CHECK(g.n == 1 && g.part[0].tile == hr::GT_BIG && g.part[0].bm == 256 && g.part[0].bn == c.bn);
        }
    }
    {   // attention: whether a block's keys are spread over wavefronts or walked in one chain
        // five pairs of the GPU test that compares the two (most blocks per pair x kv heads x 5, keys, head size), and its whole batch
        struct Spread { int n_kv, blocks, d, keys; };
        for (const Spread& c : {Spread{2, 16, 64, 2150}, Spread{4, 2, 64, 2120}, Spread{2, 5, 128, 2120}, Spread{4, 3, 128, 2150}, Spread{1, 1, 64, 2081}}) {
            CHECK(hr::attn_takes_rows(5 * c.n_kv * c.blocks, std::min(c.blocks, 16), c.d, c.keys, 256));
            CHECK(!hr::attn_takes_rows(880 * c.n_kv * c.blocks, std::min(c.blocks, 16), c.d, c.keys, 256));
        }
        CHECK(hr::attn_takes_rows(352, 4, 64, 352, 256) && !hr::attn_takes_rows(353, 4, 64, 4096, 256));
        CHECK(hr::attn_takes_rows(256, 4, 128, 256, 256) && !hr::attn_takes_rows(257, 4, 128, 4096, 256));
        CHECK(hr::attn_takes_rows(96, 1, 64, 96, 256) && !hr::attn_takes_rows(97, 1, 64, 96, 256));        // short documents
        CHECK(hr::attn_takes_rows(704, 14, 64, 512, 256) && !hr::attn_takes_rows(705, 14, 64, 512, 256));  // two blocks per wavefront in the other
    }
    {   // ... 128-wide heads, items of 5 to 8 blocks (documents in chunks of 64 tokens).  A round of workgroups: one document of 65 or of 250 tokens,
        // two of 128, not three of 64
        CHECK(hr::attn_call_takes_rows(2, 8, 8, 8, 128, 65, 256) && hr::attn_call_takes_rows(4, 8, 8, 8, 128, 250, 256));
        CHECK(hr::attn_call_takes_rows(4, 8, 8, 8, 128, 128, 256) && !hr::attn_call_takes_rows(3, 8, 8, 8, 128, 64, 256));
        // more: one document of 264 to 448 tokens, not of 449 (eight chunks), nor two of 192 or of 256
        CHECK(hr::attn_call_takes_rows(5, 8, 8, 8, 128, 264, 256) && hr::attn_call_takes_rows(6, 8, 8, 8, 128, 376, 256));
        CHECK(hr::attn_call_takes_rows(7, 8, 8, 8, 128, 448, 256) && !hr::attn_call_takes_rows(8, 8, 8, 8, 128, 449, 256));
        CHECK(!hr::attn_call_takes_rows(6, 8, 8, 8, 128, 192, 256) && !hr::attn_call_takes_rows(8, 8, 8, 8, 128, 256, 256));
        CHECK(hr::attn_takes_rows(256, 8, 128, 128, 256) && !hr::attn_takes_rows(257, 8, 128, 171, 256) && hr::attn_takes_rows(257, 8, 128, 172, 256));
        CHECK(hr::attn_takes_rows(448, 8, 128, 4096, 256) && !hr::attn_takes_rows(449, 8, 128, 4096, 256));
    }
    {   // ... and a call whose shape the spread kernel's parameters cannot hold keeps to the chain, whatever a query may be cut into
        CHECK(hr::attn_call_takes_rows(1, 1, 255, 16, 64, 4096, 256) && !hr::attn_call_takes_rows(1, 1, 256, 16, 64, 4096, 256));
        CHECK(hr::attn_call_takes_rows(5, 2, 16, 16, 64, 2150, 256) && !hr::attn_call_takes_rows(880, 2, 16, 16, 64, 2150, 256));
        CHECK(hr::rows_holds((1 << 23) - 1, 255) && !hr::rows_holds(1 << 23, 1) && !hr::rows_holds(1, 256));
    }
    {   // ... and how many of its workgroups read weights ahead
        CHECK(hr::rows_warm_wgs(544, false) == 160 && hr::rows_warm_wgs(639, false) == 160 && hr::rows_warm_wgs(640, false) == 128 && hr::rows_warm_wgs(544, true) == 128);
    }
    {   // few-rows attention: every request finds the address of the sub-tile whose size it reads (a document's fp8 page is half as long
        // as an own one), those past the last round too, at every length
        for (int n_sub = 1; n_sub <= 200; ++n_sub)
            for (int n_doc = 0; n_doc < n_sub; n_doc += n_doc < n_sub - 4 ? 3 : 1) {      // the last sub-tile holds own keys
                const int rounds = (n_sub + hr::kRoundSubs - 1) / hr::kRoundSubs;
                int at = 0;                                                               // the even round whose addresses a wavefront has
                auto right = [&](int pages, int round, int j) {                           // the kernel's request goes by the round asked for
                    const int asked = hr::rows_asked(round, rounds), there = std::min(asked * hr::kRoundSubs + j, n_sub - 1);
                    bool ok = round >= rounds || asked == round;
                    for (int side = 0; side < 2; ++side) {
                        const int lane = hr::rows_page_lane(asked, j, side), sub = hr::rows_lane_sub(pages, lane, n_sub);
                        ok = ok && lane < 64 && (lane & 1) == side && sub == there && (asked * hr::kRoundSubs + j < n_doc) == (sub < n_doc);
                    }
                    return ok;
                };
                // S wavefronts: K of the next round, requested in every round
                for (int j = 0; j < hr::kRoundSubs; ++j) CHECK(right(0, 0, j));
                for (int r = 0, nxt = 0; r < rounds; ++r) {
                    if (r & 1) at = nxt;
                    for (int j = 0; j < hr::kRoundSubs; ++j) CHECK(right(at, r + 1, j));
                    if (hr::rows_fetches_pages(r, rounds)) nxt = r + 2;
                }
                // O wavefronts: V, half a round ahead; the last round ends at its half where nothing comes behind it
                at = 0;
                for (int j = 0; j < hr::kVAhead; ++j) CHECK(right(0, 0, j));
                for (int r = 0, nxt = 0, cur = 0; r < rounds; ++r) {
                    if (r & 1) at = nxt;
                    for (int j = 0; j < hr::kRoundSubs; ++j) {
                        if (j == hr::kRoundSubs / 2 && n_sub - r * hr::kRoundSubs <= j) break;
                        CHECK(j < hr::kVAhead ? right(cur, r, j + hr::kVAhead) : right(at, r + 1, j - hr::kVAhead));
                    }
                    if (r & 1) cur = at;
                    if (hr::rows_fetches_pages(r, rounds)) nxt = r + 2;
                }
            }
        // V of an fp8 page comes in 16-byte requests of which 8 count: behind the pool's last page lie its scales
        for (int d : {64, 128}) {
            const hr::PoolLayout lay = hr::make_layout(hr_pool_cfg{1, 1, d, 16, 1, HR_FP8_E4M3});
            CHECK(lay.total_bytes >= (size_t)2 * 16 * d + 8);
        }
    }
    {   // weights read ahead by a launch's idle workgroups: never more than they can take, in order, what does not fit left out
        const int64_t q05[] = {896 * 896 * 2, 9728 * 896 * 2, 896 * 4864 * 2, 1152 * 896 * 2};      // O, gate / up, down, QKV of the 0.5B shape
        CHECK(hr::pick_weight_walks(q05, 4, 128) == 15);
        CHECK(hr::pick_weight_walks(q05, 4, 64) == 13);      // 248 pairs x 2 kv heads leave 16 of 512 workgroups, 224 pairs 64
        CHECK(hr::pick_weight_walks(q05, 4, 16) == 9);
        CHECK(hr::pick_weight_walks(q05, 4, 0) == 0 && hr::pick_weight_walks(q05, 4, -8) == 0 && hr::pick_weight_walks(q05, 0, 128) == 0);
        std::srand(17);
        for (int it = 0; it < 2000; ++it) {
            int64_t b[4], sum = 0;
            for (int64_t& x : b) x = (int64_t)128 * 64 * (1 + std::rand() % 4000);
            const int n = 1 + std::rand() % 4, wgs = 8 * (std::rand() % 17);
            const unsigned p = hr::pick_weight_walks(b, n, wgs);
            CHECK(p < 1u << n);
            for (int i = 0; i < n; ++i) {
                const bool fits = sum + b[i] <= (int64_t)wgs * hr::kWarmBytesPerWg;
                CHECK(fits == (bool)(p >> i & 1));
                if (fits) sum += b[i];
            }
        }
    }
    {   // the columns that an XCD's idle workgroups read ahead: those of its tiles, once per group of tile rows, and none of a short last
        // group, whose one or two XCDs would read the whole matrix
        for (int tiles_m = 1; tiles_m <= 70; ++tiles_m)
            for (int tiles_n : {1, 2, 3, 14, 18, 28, 76, 152}) {
                const int n_tiles = tiles_m * tiles_n, per = (n_tiles + hr::kXcds - 1) / hr::kXcds;
                for (int xcd = 0; xcd < hr::kXcds; ++xcd) {
                    const int t1 = std::min((xcd + 1) * per, n_tiles);
                    std::vector<int> want(tiles_n, 0), got(tiles_n, 0);
                    int last_group = -1, last_tn = -1;
                    for (int t = xcd * per; t < t1; ++t) {
                        const hr::TileCoord c = hr::map_tile((t - xcd * per) * hr::kXcds + xcd, tiles_m, tiles_n);
                        CHECK(c.valid && c.tm < tiles_m && c.tn < tiles_n);
                        const int group = c.tm / hr::kGroupM;
                        if (group > 0 && c.shares < hr::kAheadShares) continue;
                        if (group != last_group || c.tn != last_tn) ++want[c.tn];
                        last_group = group;
                        last_tn = c.tn;
                    }
                    int runs = 0;
                    for (int t = xcd * per; t < t1; ++runs) {
                        const hr::ColumnRun r = hr::column_run(t, t1, tiles_m, tiles_n);
                        CHECK(r.end > t && r.end <= t1 && r.c0 >= 0 && r.c0 < r.c1 && r.c1 <= tiles_n);
                        for (int c = r.c0; r.near && c < r.c1; ++c) ++got[c];
                        t = r.end;
                    }
                    CHECK(got == want && runs <= per / (hr::kGroupM * tiles_n) + 2);
                }
            }
    }
    {   // sequences with the same token string share first-layer rows: tables written into a layout of exactly the computed size
        // strings: A = {5, 6, 7}, B = {5, 6}, C = {9}; sequences A B A C B A C
        const std::vector<int32_t> lens = {3, 2, 3, 1, 2, 3, 1};
        const std::vector<int32_t> toks = {5, 6, 7, 5, 6, 5, 6, 7, 9, 5, 6, 5, 6, 7, 9};
        const int64_t n = (int64_t)lens.size(), T = (int64_t)toks.size();
        const hr::QueryShare qs = hr::make_query_share(n, lens.data(), toks.data());
        CHECK(qs.n_uniq == 6 && (int64_t)qs.rep_row.size() == 6 && (int64_t)qs.tok_src.size() == T);
        const std::vector<int32_t> want_rep = {0, 1, 2, 3, 4, 8};
        const std::vector<int32_t> want_src = {0, 1, 2, 3, 4, 0, 1, 2, 5, 3, 4, 0, 1, 2, 5};
        CHECK(qs.rep_row == want_rep && qs.tok_src == want_src);
        for (int64_t t = 0; t < T; ++t) CHECK(toks[qs.rep_row[qs.tok_src[t]]] == toks[t]);
        const hr::MetaLayout ml = hr::make_meta_layout(n, T, 4, -1, 0, 10, true);
        CHECK(ml.rep_row >= ml.tok_src + (size_t)T && ml.grp >= ml.rep_row + (size_t)T / 2 + 1 && ml.total >= ml.grp + 10);
        CHECK(qs.n_uniq * 2 <= T);                           // the tables fit the room the layout gives them
        std::vector<int32_t> meta(ml.total, -7);
        std::memcpy(meta.data() + ml.tok_src, qs.tok_src.data(), sizeof(int32_t) * qs.tok_src.size());
        std::memcpy(meta.data() + ml.rep_row, qs.rep_row.data(), sizeof(int32_t) * qs.rep_row.size());
        // equal hashes of different strings must not merge: same length, tokens differ in one place
        const std::vector<int32_t> l2 = {2, 2, 2};
        const std::vector<int32_t> t2 = {1, 2, 1, 3, 1, 2};
        const hr::QueryShare q2 = hr::make_query_share(3, l2.data(), t2.data());
        CHECK(q2.n_uniq == 4 && q2.tok_src[4] == 0 && q2.tok_src[5] == 1 && q2.tok_src[2] == 2);
        const hr::QueryShare q0 = hr::make_query_share(0, l2.data(), t2.data());
        CHECK(q0.n_uniq == 0 && q0.tok_src.empty());
        // workspace: the split form doubles the activation buffers, the shared form adds fp32 rows for half the tokens
        hr_model_cfg mc{2, 256, 4, 2, 64, 320, 500, 1, 2, HR_BF16, 10000.0f, 1e-6f};
        const hr::Workspace w0 = hr::make_workspace(mc, 4, 100, 3, false), w1 = hr::make_workspace(mc, 4, 100, 3, false, -1, 0, 0, true),
                            w2 = hr::make_workspace(mc, 4, 100, 3, false, -1, 0, 0, false, true);
        CHECK(w1.total > w0.total && w2.total > w0.total && w1.off_kvlo >= w1.off_v && w1.off_o > w1.off_kvlo && w0.off_o == w0.off_kvlo);
    }
    std::printf("host logic clean under sanitizers\n");
    return 0;
}

// Device tables of a plan: the re-layout segment list, the split-KV decode
// work items and the prefill tile schedules (packed and padded).  Host only.
//
// Packed prefill (Sec. 3.1, execution domain = union of valid query-key
// regions): query tiles are cut from the packed token stream of each group
// and may span requests; a tile lists only the key tiles that hold at least
// one unmasked pair for it, and each key tile says per wave (32 query rows)
// whether that wave skips it, computes it with the mask, or computes it
// without any mask.  With an even number of query heads per KV head a
// workgroup takes the rows of several heads of one request instead
// (emit_head_tiles), but for launches that leave units idle and for eight
// waves with two or six heads per KV head.
#include <algorithm>
#include <cmath>
#include <numeric>

#include "plan.h"

namespace pk {

namespace {

struct Builder {
    std::vector<int32_t>& host;
    explicit Builder(std::vector<int32_t>& h) : host(h) {}
    TableRef add(const std::vector<int32_t>& v) {
        TableRef r;
        host.resize((host.size() + 63) / 64 * 64, 0);
        r.offset = host.size() * sizeof(int32_t);
        r.count = v.size();
        host.insert(host.end(), v.begin(), v.end());
        return r;
    }
    // Room for a table that the caller fills by index (the pointer is good until the next table).
    int32_t* room(size_t count, TableRef& r) {
        host.resize((host.size() + 63) / 64 * 64, 0);
        r.offset = host.size() * sizeof(int32_t);
        r.count = count;
        host.resize(host.size() + count);
        return host.data() + (host.size() - count);
    }
};

// ---- re-layout -------------------------------------------------------------
void build_reorg(const pk_plan& plan, Builder& b, DeviceTables& t) {
    struct Seg { int64_t dst0; int32_t ntok, req, src0; };
    std::vector<Seg> segs;
    segs.reserve(static_cast<size_t>(plan.n));
    for (const Group& g : plan.groups) {
        for (const Node& nd : g.nodes)                            // a shared segment once, via its lowest request
            segs.push_back({g.buf_base + nd.off, nd.len, nd.reqs[0], nd.start});
        for (const Member& m : g.members)
            if (m.lq > 0) segs.push_back({g.buf_base + m.suffix_off, m.lq, m.req, m.shared});
    }
    auto before = [](const Seg& x, const Seg& y) { return x.dst0 < y.dst0; };
    if (!std::is_sorted(segs.begin(), segs.end(), before)) std::sort(segs.begin(), segs.end(), before);   // (without shared segments they are)
    int32_t* flat = b.room(segs.size() * 4, t.reorg_seg);
    for (const Seg& s : segs) {
        *flat++ = static_cast<int32_t>(s.dst0); *flat++ = s.ntok;
        *flat++ = s.req; *flat++ = s.src0;
    }
    const int64_t nb = plan.buf_tokens / kDecodeBlock;
    int32_t* first = b.room(static_cast<size_t>(nb), t.reorg_blk_first);
    size_t cur = 0;
    for (int64_t blk = 0; blk < nb; ++blk) {
        const int64_t t0 = blk * kDecodeBlock;
        while (cur < segs.size() && segs[cur].dst0 + segs[cur].ntok <= t0) ++cur;
        first[blk] = static_cast<int32_t>(cur);
    }
    t.n_reorg_seg = static_cast<int32_t>(segs.size());
}

// ---- decode ----------------------------------------------------------------
// Split length for a batch whose (work item, KV head) pairs are served by a workgroup of four waves each, 0 where a wave
// each is the better choice.  A workgroup streams an item 3 to 4 times as fast as a wave does, so that most requests need no
// split, and it merges in the same launch what is split.  With waves / with workgroups (us, buffers that repeat; both sides
// with the better split): one request of 500 tokens 8.9 / 6.3, four of 300..3000 11.5 / 11.3 and 10.8 / 9.5 (two cards), 24 of 1500 26.3 / 23.4, 59 of 428
// with 28/4 heads 13.3 / 9.3, 480 lognormal around 1000 with 64/8 heads 418 / 391, 200 around 700 with head dimension 64
// 73.4 / 69.7, 256 of 32..32768 200 / 192, 480 rows up to 65536 2860 / 2590.  Waves stay
//   - for items with rows of several requests or more than 16 rows (the kernel has one column tile of rows and merges one request);
//   - for many short requests, where the waves of a workgroup get a tile or two each: 600 of 20..200 tokens with 28/4
//     heads 29.0 / 34.4, 1000 of 128 with 4/1 heads 10.9 / 14.8, 300 of 200 41.7 / 44.4; 305 around 278 with head
//     dimension 64 31.8 / 30.4, 591 of 300..400 with 4/1 heads 22.1 / 19.9;
//   - for requests of at most four tiles, which a wave does not split either: 78 of 8..32 tokens 5.4 / 7.7;
//   - for short launches with many partial results to a request, which a merge of sixteen waves reads faster: one of
//     11513 tokens and 32/8 heads (20 partial results) 13.9 / 14.5, of 8799 and 16/2 heads (23) 10.0 / 10.8; one of 16000
//     and 32/8 heads (23) 16.1 / 15.6, of 32768 (20) 27.9 / 25.1.  Merged rows count as well: one workgroup reads the partial results of all
//     query heads of a KV head.  One of 4000 tokens (11 partial results): 32/8 heads 9.3 / 9.9 and 8/2 heads 9.3 / 8.1, 64/8 9.5 / 10.4, 64/4
//     9.7 / 11.2, 32/2 9.2 / 11.2; two of 3000 and 2500 (8): 16/2 9.4 / 8.5, 32/2 9.0 / 9.0, 64/4 9.0 / 9.8; one of 1500 (4) 64/8 9.4 / 8.8, 64/4 9.0 / 9.8,
//     16/1 9.6 / 8.4; eight of 3000 (5) 64/4 14.3 / 13.1.  (From a captured graph, where a second launch costs 2 us less, waves are ahead from two partial results on.)
// The split is the one with the least estimated time: bytes at the rate of the whole chip, a start and an end of each workgroup,
// and the longest item alone for as long as its fair share of the other workgroups' time does not cover it.  The estimate
// picks within 2 % of the best split on average over 57 batches of 1..1000 requests (10 % at worst).  No split is shorter
// than the one for waves (`from`): there are never more work items and partial results than with that.  None is longer than
// 8 MiB of a KV head: beside the prefill tiles of a mixed step a workgroup is slow, and whole sequences of 65536
// tokens keep the chip when everything else is done (12.52 instead of 12.23 ms for 32 chunks and 480 rows of a 70B-shaped
// layer; with the limit as fast as with waves).
int64_t group_split(const pk_plan& plan, int r, int Hkv, int d, int num_cus, int64_t from) {
    std::vector<int32_t> blocks;
    blocks.reserve(static_cast<size_t>(plan.n));
    int64_t total = 0;
    int32_t longest = 0;
    auto segment = [&](int32_t len) {
        const int32_t k = static_cast<int32_t>((static_cast<uint32_t>(len) + kDecodeBlock - 1) / kDecodeBlock);
        if (k > 0 || plan.headroom > 0) blocks.push_back(std::max(k, 1));
        total += k;
        longest = std::max(longest, k);
    };
    for (const Group& g : plan.groups) {
        for (const Node& nd : g.nodes) {
            if (nd.reqs.size() > 1) return 0;
            segment(nd.len);
        }
        for (const Member& m : g.members) segment(m.lq);
    }
    if (longest <= 4) return 0;
    // in nanoseconds (a tile of head dimension 64 has half the bytes): a tile at the rate of the whole chip and
    // of one workgroup, a workgroup's start and end, a merge
    const double scale = d / 128.0;
    const double all = 3.2 * scale, alone = 530 * scale, fixed = 6.5 * (1 + scale), merge = 2000;
    const int64_t slots = static_cast<int64_t>(2 * num_cus / scale);
    double best = 0;
    int64_t split = 0, best_wgs = 0, best_parts = 0;
    // (`from` is at most 8192 tokens and sp ends at 410 tiles of 16 KiB or so: 32 bits; most requests are whole, without a division)
    for (int32_t sp = std::max(static_cast<int32_t>(from / kDecodeBlock), static_cast<int32_t>(12 / scale)); ; sp = sp * 5 / 4) {
        int64_t items = 0;
        int32_t most = 0, parts = 1;
        for (const int32_t b : blocks) {
            if (b <= sp) {
                ++items;
                most = std::max(most, b);
                continue;
            }
            const int32_t pieces = static_cast<int32_t>((static_cast<uint32_t>(b) + static_cast<uint32_t>(sp) - 1) / static_cast<uint32_t>(sp));
            items += pieces;
            parts = std::max(parts, pieces);
            most = std::max(most, (b + pieces - 1) / pieces);
        }
        const double wgs = static_cast<double>(items) * Hkv, work = static_cast<double>(total) * Hkv;
        const double share = work / std::min(wgs, static_cast<double>(slots)), per_cu = wgs / num_cus;
        // a compute unit streams no faster with two workgroups than with one: 24 requests of 1500 tokens in 192 workgroups 23.9 us,
        // in 384 29.1, in 576 30.3; 4 of 65536 in 192 150 us, in 256 160, in 352 175, in 512 165
        const double uneven = per_cu > 1 ? 0.5 + 0.5 * std::ceil(per_cu) / per_cu : 1.0;
        const double t = (work * all + wgs * fixed) * std::max(uneven, alone / all / wgs) + std::max(0.0, static_cast<double>(most) - share) * alone +
                         (items > plan.n ? merge : 0.0);
        if (split == 0 || t < best) { best = t; split = int64_t{sp} * kDecodeBlock; best_wgs = items * Hkv; best_parts = parts; }
        if (sp >= longest || sp * scale >= 410) break;       // (the next one could exceed 512 tiles of 16 KiB)
    }
    if (best_wgs > 3 * num_cus && total * Hkv < 8 * best_wgs) return 0;
    if (best_parts > 32 || (best_parts > 16 && best < 15000) || (best_parts * r > 64 && best < 12500)) return 0;
    return split;
}

// Split length of the shared segments of a batch whose items have a wave each.  A piece of a shared segment leaves a partial result for every one of up
// to 32 rows (16 KiB with d = 128, written and read again, beside 16 KiB of K/V a tile), and a wave alone takes 1.6 us (d = 64: 1.3) for a tile of such a piece: short pieces
// cost the memory system, long ones outlast the launch.  The split of the suffixes knows neither: it is the shortest, 128 tokens, for small batches, and 2048 where the suffixes
// alone are more waves than the chip holds.  Taken is the length with the least estimated time: bytes (K/V, of which the pieces of more requests than
// one item takes read half again, and partial results twice) at 5.9 TB/s and 4.2 us for 2048 waves (half of it with d = 64, where twice as many run at a
// time), or the longest item alone, whichever is more, and a sixth of the other.  us, with the split of the suffixes / with this one: 182 requests of 33 tokens, 11 segments of 2000 below one of 2843 with
// 16/16 heads 77.5 / 58.0 (2048 and 512 tokens), 279 of 63 with 34 of 876 62.2 / 47.8, 321 of 55 with 40 of 1259 below 1667 88 / 73; 40 of 350 with 20 of 2743 and 16/2 heads 20.5 / 16.5 (128 and
// 256), 268 of 130 with 67 of 1880 41.6 / 36.2.  The constants are fitted to 92 random batches at eleven lengths each: 1.03 times as fast as with one split for
// all, with the best length of each 1.049.  Estimated gains of less than 3 %, 5 for shorter pieces, are left: of 58 other batches 23 had such, and six of those lost 2 to 11 %.
// Where the length is changed, 80 other batches are 1.11 times as fast (0.945 to 1.79; eight of them more than 2 % slower).
int64_t shared_split(const pk_plan& plan, int Hq, int Hkv, int d, int max_members, int64_t split) {
    const double row_bytes = 4.0 * d * Hq, token_bytes = 4.0 * d * Hkv;
    struct Shared { int32_t blocks, requests, chunks; };
    std::vector<Shared> shared;
    double waves = 0, bytes = 0;                   // of what has one request
    int32_t longest = 0, longest_shared = 0;
    const int32_t own = static_cast<int32_t>(split / kDecodeBlock);
    auto blocks_of = [](int32_t len) { return static_cast<int32_t>((static_cast<uint32_t>(len) + kDecodeBlock - 1) / kDecodeBlock); };
    auto single = [&](int32_t len) {
        const int32_t blocks = blocks_of(len), pieces = std::max(1, blocks <= own ? 1 : (blocks + own - 1) / own);
        waves += pieces;
        bytes += len * token_bytes + 2 * pieces * row_bytes;
        longest = std::max(longest, (blocks + pieces - 1) / pieces);
    };
    for (const Group& g : plan.groups) {
        for (const Node& nd : g.nodes) {
            const int32_t n = static_cast<int32_t>(nd.reqs.size());
            if (n < 2) { single(nd.len); continue; }
            const int32_t blocks = blocks_of(nd.len), chunks = (n + max_members - 1) / max_members;
            shared.push_back({blocks, n, chunks});
            bytes += nd.len * token_bytes * (1 + 0.5 * (chunks - 1));
            longest_shared = std::max(longest_shared, blocks);
        }
        for (const Member& m : g.members) single(m.lq);
    }
    if (longest_shared * kDecodeBlock <= 128) return split;            // (whole at any length)
    auto time = [&](int32_t sp) {
        double w = waves, b = bytes;
        int32_t most = 0;
        for (const Shared& x : shared) {
            const int32_t pieces = x.blocks <= sp ? 1 : (x.blocks + sp - 1) / sp;
            w += pieces * x.chunks;
            b += 2.0 * pieces * x.requests * row_bytes;
            most = std::max(most, (x.blocks + pieces - 1) / pieces);
        }
        const double chip = b / 5.9e6 + (d <= 64 ? 2.1 : 4.2) / 2048 * w * Hkv, alone = std::max(1.56 * most, 1.05 * longest) * (d <= 64 ? 0.85 : 1.0);
        return std::max(chip, alone) + 0.16 * std::min(chip, alone);
    };
    const double one = time(own);
    double best = one;
    int32_t taken = own;
    for (int32_t sp = 4; ; sp = sp * 3 / 2) {      // 128 to 2016 tokens
        const double t = time(sp);
        if (t < best && t < one * (sp < own ? 0.95 : 0.97)) { best = t; taken = sp; }
        if (sp >= longest_shared || sp >= 63) break;
    }
    return int64_t{taken} * kDecodeBlock;
}

void build_decode(const pk_plan& plan, int Hq, int Hkv, int d, int dtype, int num_cus, bool may_choose, Builder& b, DeviceTables& t) {
    const int r = Hq / Hkv;
    const int max_members = std::max(1, kDecodeMaxRows / r);
    // split length: about 1500 waves (work items x KV heads) keep enough loads in flight to fill
    // the memory system (each has 32 KiB outstanding); beyond that, longer items mean fewer
    // partial results to write and merge
    const int64_t share = plan.unique_tokens * Hkv / 1536;
    auto whole_blocks = [](int64_t tokens) { return (tokens + kDecodeBlock - 1) / kDecodeBlock * kDecodeBlock; };
    int64_t split = std::min<int64_t>(std::max<int64_t>(whole_blocks(share), 128), 2048);
    {
        // All waves of the launch should be resident at once (a second, partly filled round of
        // waves is a tail as long as a whole item): 8 per CU fit with the registers of head dimension
        // 128, 16 with those of 64.  Short suffixes cost an item each whatever the split, so the items are
        // counted for the candidate and the split is raised until they fit -- but not so far that
        // one wave alone (20 GB/s, half of it with head dimension 64) takes longer than half the launch.
        // 61 requests of 346..65536 tokens: 2048 tokens (3264 waves) 521 us, 4000 (1776 waves) 483 us,
        // 8192 486 us.  Batches with too many requests to fit gain from neither (480 rows: 2048 tokens,
        // 256 requests of 32..32768: 1632 202.8 us, 2048 200.9, 4096 204.7, 8192 224).
        bool wide = false;                         // items with more than 16 query rows: fewer registers to spare
        for (const Group& g : plan.groups)
            for (const Node& nd : g.nodes) wide = wide || static_cast<int>(std::min<size_t>(nd.reqs.size(), max_members)) * r > 16;
        const int64_t capacity = static_cast<int64_t>(d <= 64 && !wide ? 16 : 8) * num_cus * 9 / 10;
        // (no division where it is one: most requests are whole)
        auto pieces_of = [&](int64_t len, int64_t sp) { return len <= 0 ? int64_t{0} : whole_blocks(len) <= sp ? int64_t{1} : (whole_blocks(len) + sp - 1) / sp; };
        auto fits = [&](int64_t sp, int64_t waves) {
            int64_t c = 0;
            for (const Group& g : plan.groups) {
                for (const Node& nd : g.nodes)
                    c += pieces_of(nd.len, sp) * static_cast<int64_t>((nd.reqs.size() + max_members - 1) / max_members);
                for (const Member& m : g.members) c += std::max<int64_t>(pieces_of(m.lq, sp), plan.headroom > 0 ? 1 : 0);
            }
            return c * Hkv <= waves;
        };
        const int64_t longest = std::min<int64_t>(std::max<int64_t>(whole_blocks(share * 5 / (d <= 64 ? 4 : 2)), split), 8192);
        // from `from` in steps of a quarter up to `most`, until `waves` waves are enough
        auto raise = [&](int64_t from, int64_t most, int64_t waves) {
            while (from < most && !fits(from, waves)) from = std::min(most, whole_blocks(from * 5 / 4));
            return from;
        };
        // where not even that fits, the even share and a quarter (the share / that / twice the share: 300 requests of
        // 100..700 tokens 81.7 / 77.8 / 77.8 us, 260 of 100..2500 213.6 / 210.9 / 206.7, 400 lognormal around 300 160.5 /
        // 160.0 / 163.2, 550 around 200 with head dimension 64 96.6 / 97.2 / 99.6); and in every case no more partial results
        // than two rounds of waves leave (the fixed scratch of pk_packed_decode_attn_static holds those)
        const int64_t two_rounds = raise(split, 2048, static_cast<int64_t>(wide ? 8 : 16) * num_cus * 9 / 10);
        const int64_t raised = raise(split, longest, capacity);
        split = std::max(two_rounds, fits(raised, capacity) ? raised : std::min<int64_t>(2048, whole_blocks(split * 5 / 4)));
    }
    split = whole_blocks(split);
    const bool may = may_choose && dtype == PK_BF16 && r <= 16;
    int64_t by_group = may ? group_split(plan, r, Hkv, d, num_cus, split) : 0;
    if (plan.tune_decode_split > 0) {              // pk_plan_tune (profiling sweeps): another split for the same kernel
        split = whole_blocks(plan.tune_decode_split);
        if (by_group > 0) by_group = split;
    }
    int64_t shared = split;                        // split of the shared segments
    if (may && by_group == 0 && plan.tune_decode_split == 0) {
        bool any = false;
        for (const Group& g : plan.groups) any = any || !g.nodes.empty();
        if (any) shared = shared_split(plan, Hq, Hkv, d, max_members, split);
    }

    struct Segment { int64_t a, e; const int32_t* reqs; int32_t n_reqs; bool suffix; };   // (reqs point into the plan)
    std::vector<Segment> segments;
    segments.reserve(static_cast<size_t>(plan.n));
    std::vector<int32_t> req_seg(static_cast<size_t>(plan.n) * 4, 0);
    std::vector<std::vector<int32_t>> chain_of(static_cast<size_t>(plan.n));
    struct Piece { int32_t off; int32_t node, member; };
    std::vector<Piece> pieces;
    for (const Group& g : plan.groups) {
        // work items in layout order: a shared segment attends for every request below it
        if (g.nodes.empty()) {                     // (members are in that order)
            for (const Member& mm : g.members) {
                segments.push_back({g.buf_base + mm.suffix_off, g.buf_base + mm.suffix_off + mm.lq, &mm.req, 1, true});
                int32_t* rs = &req_seg[static_cast<size_t>(mm.req) * 4];
                rs[0] = static_cast<int32_t>(g.buf_base + mm.prefix_off); rs[1] = mm.lp;
                rs[2] = static_cast<int32_t>(g.buf_base + mm.suffix_off); rs[3] = mm.lq;
            }
            continue;
        }
        pieces.clear();
        for (size_t k = 0; k < g.nodes.size(); ++k) pieces.push_back({g.nodes[k].off, static_cast<int32_t>(k), -1});
        for (size_t k = 0; k < g.members.size(); ++k) pieces.push_back({g.members[k].suffix_off, -1, static_cast<int32_t>(k)});
        std::stable_sort(pieces.begin(), pieces.end(), [](const Piece& x, const Piece& y) { return x.off < y.off; });
        for (const Piece& pc : pieces) {
            if (pc.node >= 0) {
                const Node& nd = g.nodes[static_cast<size_t>(pc.node)];
                segments.push_back({g.buf_base + nd.off, g.buf_base + nd.off + nd.len, nd.reqs.data(), static_cast<int32_t>(nd.reqs.size()), false});
                continue;
            }
            const Member& mm = g.members[static_cast<size_t>(pc.member)];
            segments.push_back({g.buf_base + mm.suffix_off, g.buf_base + mm.suffix_off + mm.lq, &mm.req, 1, true});
            int32_t* rs = &req_seg[static_cast<size_t>(mm.req) * 4];
            rs[0] = static_cast<int32_t>(g.buf_base + mm.prefix_off); rs[1] = mm.lp;
            rs[2] = static_cast<int32_t>(g.buf_base + mm.suffix_off); rs[3] = mm.lq;
            std::vector<int32_t>& ch = chain_of[static_cast<size_t>(mm.req)];
            for (int32_t k = mm.node; k >= 0; k = g.nodes[static_cast<size_t>(k)].parent) {
                ch.push_back(g.nodes[static_cast<size_t>(k)].len);            // reversed below: innermost first here
                ch.push_back(static_cast<int32_t>(g.buf_base + g.nodes[static_cast<size_t>(k)].off));
            }
            std::reverse(ch.begin(), ch.end());                   // (offset, tokens) pairs, outermost first
        }
    }
    std::vector<int32_t> chain_start(static_cast<size_t>(plan.n) + 1, 0), chain;
    for (int32_t i = 0; i < plan.n; ++i) {
        chain.insert(chain.end(), chain_of[static_cast<size_t>(i)].begin(), chain_of[static_cast<size_t>(i)].end());
        chain_start[static_cast<size_t>(i) + 1] = static_cast<int32_t>(chain.size() / 2);
    }
    t.dec_req_seg = b.add(req_seg);
    t.dec_chain_start = b.add(chain_start);
    t.dec_chain = b.add(chain);

    struct Item { int64_t a, e; const int32_t* reqs; int32_t n_reqs; bool grows; };
    // suffix: the segment is a request's private suffix; its last item is marked so that the
    // kernel extends it by the tokens appended into the headroom since the plan was made (an
    // empty suffix with headroom still gets an item for them)
    auto cut = [&](int64_t split) {
        std::vector<Item> items;
        items.reserve(segments.size() + segments.size() / 4);
        for (const auto& [a, e, reqs, n_reqs, suffix] : segments) {
            if (e <= a) {
                if (suffix && plan.headroom > 0) items.push_back({a, a, reqs, n_reqs, true});
                continue;
            }
            // the fewest pieces of at most `split` tokens, all of (nearly) the same length: a full-length
            // piece next to a short remainder would set the pace of the launch for little work
            const int64_t a_blk = a / kDecodeBlock * kDecodeBlock;
            const int64_t blocks = (e - a_blk + kDecodeBlock - 1) / kDecodeBlock;
            const int64_t most = n_reqs > 1 ? shared : split;
            const int64_t pieces = blocks * kDecodeBlock <= most ? 1 : (blocks * kDecodeBlock + most - 1) / most;
            const int64_t piece = (pieces == 1 ? blocks : (blocks + pieces - 1) / pieces) * kDecodeBlock;
            for (int32_t m0 = 0; m0 < n_reqs; m0 += max_members)
                for (int64_t p0 = a_blk; p0 < e; p0 += piece)
                    items.push_back({std::max(a, p0), std::min(e, p0 + piece), reqs + m0, std::min(n_reqs - m0, max_members),
                                     suffix && p0 + piece >= e});
        }
        return items;
    };
    std::vector<int32_t> n_items_of(static_cast<size_t>(plan.n), 0);
    DeviceTables::DecodeSched& s = t.dec;
    s.chosen = by_group > 0 || shared != split;
    if (s.chosen) {                                // (a wave each and one split: counted without building the items)
        for (const Segment& g : segments) {
            if (g.e <= g.a && !(g.suffix && plan.headroom > 0)) continue;
            const int64_t blocks = g.e <= g.a ? 1 : (g.e - g.a / kDecodeBlock * kDecodeBlock + kDecodeBlock - 1) / kDecodeBlock, pieces_at = split / kDecodeBlock;
            // (whole pieces of equal length: fewer than pieces_of would say where the length is rounded up)
            const int64_t pieces = blocks <= pieces_at ? 1 : (blocks + pieces_at - 1) / pieces_at, piece = (blocks + pieces - 1) / pieces;
            const int32_t k = static_cast<int32_t>((blocks + piece - 1) / piece);
            s.wave_items += k * ((g.n_reqs + max_members - 1) / max_members);
            s.wave_members += k * g.n_reqs;
            for (int32_t y = 0; y < g.n_reqs; ++y) n_items_of[static_cast<size_t>(g.reqs[y])] += k;
        }
        for (int32_t& c : n_items_of) {
            s.wave_parts += c > 1 ? c : 0;
            c = 0;
        }
        if (by_group > 0) split = by_group;
    }
    s.split_tokens = static_cast<int32_t>(split);
    s.group = by_group > 0;
    const std::vector<Item> items = cut(split);
    // items with more than 16 query rows first (they run the two-column-tile kernel), then
    // the others; inside each class the longest first (stable: deterministic)
    auto wide = [&](const Item& it) { return it.n_reqs * r > 16; };
    // (as one number: the class, the length from the longest down, the item)
    std::vector<uint64_t> order(items.size());
    for (size_t x = 0; x < items.size(); ++x) {
        const uint64_t length = static_cast<uint64_t>(items[x].e - items[x].a);        // (under 2^31)
        order[x] = (wide(items[x]) ? uint64_t{0} : uint64_t{1} << 63) | (0x7FFFFFFF - length) << 32 | x;
        s.n_wide += wide(items[x]) ? 1 : 0;
    }
    std::sort(order.begin(), order.end());
    // Partial slots: the slots of one request are consecutive (the merge streams them without
    // indirection); a request covered by a single work item gets no slot: that item writes the
    // final output itself (slot -1).
    std::vector<int32_t> start(static_cast<size_t>(plan.n) + 1, 0);
    size_t n_members = 0;
    for (const Item& it : items) {
        n_members += static_cast<size_t>(it.n_reqs);
        for (int32_t x = 0; x < it.n_reqs; ++x) ++n_items_of[static_cast<size_t>(it.reqs[x])];
    }
    int32_t n_parts = 0;
    for (int32_t i = 0; i < plan.n; ++i) {
        start[static_cast<size_t>(i)] = n_parts;
        if (n_items_of[static_cast<size_t>(i)] > 1) n_parts += n_items_of[static_cast<size_t>(i)];
    }
    start[static_cast<size_t>(plan.n)] = n_parts;
    s.n_items = static_cast<int32_t>(items.size());
    s.n_members = static_cast<int32_t>(n_members);
    s.n_parts = n_parts;
    for (int32_t c : n_items_of) s.max_parts = std::max(s.max_parts, c > 1 ? c : 0);
    auto item_at = [&](size_t x) -> const Item& { return items[order[x] & 0xFFFFFFFFu]; };
    int32_t first = 0;
    int32_t* w = b.room(items.size() * 8, s.items);
    for (size_t x = 0; x < items.size(); ++x, w += 8) {
        const Item& it = item_at(x);
        w[0] = static_cast<int32_t>(it.a); w[1] = static_cast<int32_t>(it.e); w[2] = first; w[3] = it.n_reqs;
        w[4] = it.grows ? 1 : 0; w[5] = w[6] = w[7] = 0;
        first += it.n_reqs;
    }
    w = b.room(n_members, s.members);
    for (size_t x = 0; x < items.size(); ++x) w = std::copy(item_at(x).reqs, item_at(x).reqs + item_at(x).n_reqs, w);
    std::vector<int32_t> next_slot(start.begin(), start.end() - 1);
    w = b.room(n_members, s.member_slot);
    for (size_t x = 0; x < items.size(); ++x)
        for (int32_t y = 0; y < item_at(x).n_reqs; ++y) {
            const size_t rq = static_cast<size_t>(item_at(x).reqs[y]);
            *w++ = n_items_of[rq] > 1 ? next_slot[rq]++ : -1;
        }
    s.req_part_start = b.add(start);
    if (s.group) s.arrived = b.add(std::vector<int32_t>(static_cast<size_t>(plan.n) * Hkv, 0));
}

// ---- prefill ---------------------------------------------------------------
// Key tiles of so many keys (fewer than 2^31, and up to a query tile more).
int32_t key_tiles_to(int64_t keys) { return static_cast<int32_t>((static_cast<uint32_t>(keys) + kPrefillBN - 1) / kPrefillBN); }

struct RowRun { int32_t begin, count, req, t; };   // tile rows [begin, begin + count) are request req's query rows t, t + 1, ...

// Flat arrays of a schedule under construction (tiles in construction order).
struct SchedBuild {
    std::vector<int32_t> runs;                    // (first tile row, its Q row, lo, its hi) of every run of rows of one request
    std::vector<int32_t> run_first, n_runs;       // per tile
    std::vector<int32_t> kv;                      // (k_start, info) pairs of all tiles
    std::vector<int32_t> kv_first, n_kv, n_rows;  // per tile
    std::vector<int64_t> weight;                  // active (wave, key tile) pairs per tile
    int64_t issued = 0;
    void reserve(size_t tiles, size_t n, size_t key_tiles) {
        runs.reserve(4 * n);
        kv.reserve(2 * key_tiles);
        for (std::vector<int32_t>* v : {&run_first, &n_runs, &kv_first, &n_kv, &n_rows}) v->reserve(tiles);
        weight.reserve(tiles);
    }
};

// Appends one query tile (the runs cover rows 0..nrows) and its key-tile list.  all_waves: the padded
// schedule never lets a wave skip.
void add_tile(const pk_plan& plan, const std::vector<int64_t>& q_start,
              const std::vector<int64_t>& kv_start, const RowRun* tile_runs, const RowRun* tile_runs_end,
              bool all_waves, SchedBuild& sb) {
    constexpr int BM = kPrefillBM, BN = kPrefillBN, WR = 32, NW = BM / WR;
    sb.run_first.push_back(static_cast<int32_t>(sb.runs.size() / 4));
    const size_t kv0 = sb.kv.size();
    const int nrows = tile_runs_end[-1].begin + tile_runs_end[-1].count;
    int64_t weight = 0;
    for (const RowRun* x = tile_runs; x < tile_runs_end; ++x) {
        const RowRun& run = *x;
        const int32_t rq = run.req;
        const int i = run.begin, j = run.begin + run.count;
        const int64_t ks0 = kv_start[rq];
        const int64_t ctx = plan.kv_lens[rq] - plan.q_lens[rq];
        const int64_t hi0 = ks0 + ctx + run.t + 1;                       // hi of the run's first row
        const int64_t kend = hi0 + run.count - 1;                        // and of its last
        // row x of the run is Q row q_start + t + (x - i) and sees the keys [ks0, ks0 + ctx + t + 1 + (x - i))
        const int32_t entry[4] = {i, static_cast<int32_t>(q_start[rq] + run.t), static_cast<int32_t>(ks0), static_cast<int32_t>(hi0)};
        sb.runs.insert(sb.runs.end(), entry, entry + 4);
        // per wave: its rows inside the run, and whether it holds rows of no other request (waves without rows
        // of the run take no part in its key tiles)
        const int w_first = all_waves ? 0 : i / WR, w_end = all_waves ? NW : (j - 1) / WR + 1;
        int wa[NW], wb[NW];
        bool pure[NW];
        for (int w = w_first; w < w_end; ++w) {
            wa[w] = std::max(i, w * WR);
            wb[w] = std::min(j, (w + 1) * WR);
            pure[w] = i <= w * WR && std::min(nrows, (w + 1) * WR) <= j;
        }
        for (int64_t ks = ks0; ks < kend; ks += BN) {
            const int64_t ke = std::min(kend, ks + BN);
            int32_t flags = 0;
            for (int w = w_first; w < w_end; ++w) {
                int code = 0;
                if (wa[w] < wb[w] && ks < hi0 + (wb[w] - 1 - i)) {
                    const bool below = ke <= hi0 + (wa[w] - i);
                    code = (pure[w] && below && ke - ks == BN) ? 2 : 1;
                } else if (all_waves) {
                    code = 1;
                }
                weight += code != 0;
                flags |= code << (2 * w);
            }
            if (flags == 0) continue;
            sb.kv.push_back(static_cast<int32_t>(ks));
            sb.kv.push_back(static_cast<int32_t>(ke - ks) | (flags << 8));
        }
    }
    sb.issued += weight * WR * BN;
    sb.kv_first.push_back(static_cast<int32_t>(kv0 / 2));
    sb.n_kv.push_back(static_cast<int32_t>((sb.kv.size() - kv0) / 2));
    sb.n_rows.push_back(nrows);
    sb.n_runs.push_back(static_cast<int32_t>(sb.runs.size() / 4) - sb.run_first.back());
    sb.weight.push_back(weight);
}

void add_idle_tile(SchedBuild& sb) {               // padded grid slot of a request without that many tiles
    sb.run_first.push_back(static_cast<int32_t>(sb.runs.size() / 4));
    sb.n_runs.push_back(0);
    sb.kv_first.push_back(static_cast<int32_t>(sb.kv.size() / 2));
    sb.n_kv.push_back(0); sb.n_rows.push_back(0); sb.weight.push_back(0);
}

// Which of the two bodies a prefill launch takes: prefill_few_body.hip.h (true) or prefill_body.hip.h; tiles: query tiles of 128 rows that
// have key tiles, whatever tiles the launch has.
// The pipeline of the latter costs a first and a last turn of every workgroup and more issued instructions, and saves energy:
// it is the faster one where power holds the clock down, in launches of some 200 us and more, and where a wave has a long list
// to go through.  So the line is drawn by the total of key tiles times the length of a list, per compute unit.  us, pipeline / other body:
//   d = 128, lists of about 2 tiles, 64 x 200 tokens and 32 heads 80.7 / 77.0, 256 x 130 and 64 heads 431 / 404, 512 x 300 2015 / 1997;
//   5 to 10 tiles: 16 x 512 and 32 heads 46.6 / 44.7, 16 x 1024 180.7 / 174.6, twice that (75000 key tiles) 1 % the other way;
//   17 tiles: 24 x 128 behind 1000 and 32 heads 62.9 / 61.4, 64 x 128 the same; 33 tiles: 14 x 128 behind 2000 65.1 / 65.6,
//   16 x 128 68.1 / 70.7, 1 x 1024 behind 8192 (256 workgroups of 136 tiles) 152.5 / 155.2;
//   d = 64, about 2 tiles: 64 x 200 and 64 heads 83.7 / 77.0, 256 x 130 247 / 225, 512 x 300 1144 / 1102; 5 to 9 tiles: 21 x 768 and 32
//   heads 81.2 / 77.6, 32 x 1024 and 16 heads 105.2 / 101.9; 17 tiles: 24 x 128 behind 1000 and 32 heads 38.3 / 37.9, 64 x 128
//   93.4 / 90.5, 8 x 2048 (70000) 1 % the other way at 64 heads; 33 tiles: 14 x 128 behind 2000 43.9 / 43.2, 16 x 128 46.3 / 46.1.
// Over 680 such shapes the choice is within 4 % of the better one, but for prompts of exactly 32 rows, four to a tile (64 x 32
// 15.1 / 15.7 us, d = 64 17.2 / 18.4), whose waves skip three of the four key tiles in the list.  (With query tiles of several heads, 170
// shapes: 0.9 % more than the better one on average, 5 % at most but for three; the best line there would take 0.6 %.)
// Below one workgroup per unit (with d = 64 one and a half: three share a unit) the other body is the better one with any list: 7 x 57 rows
// behind 2500 tokens with 32 heads (224 workgroups) 43.9 / 40.4 and 33.1 / 32.4, 1 x 512 behind 8192 (128) 142.4 / 134.3 and
// 115.1 / 106.5, 1 x 64 behind 8000 with 8 heads (8) 124.5 / 114.0 and 94.0 / 91.8.
// The prefill half of a mixed step follows the same line, so that its results are those of the prefill call bit for bit, but for lists that only the call has in pieces (64 x 200 with 32
// heads and 32 decode rows of 500 tokens 87.2 / 81.8, 8 x 1024 and 256 of 700 178 / 173; d = 64 98.7 / 94.5).
bool light_launch(int64_t tiles, int64_t key_tiles, int Hq, int d, int num_cus) {
    if (tiles == 0) return true;
    const int64_t wgs = tiles * Hq;
    if (d == 64 ? 2 * wgs < 3 * num_cus : wgs < num_cus) return true;
    if (key_tiles < (d == 64 ? 8 : 5) * tiles) return true;
    const double list = static_cast<double>(key_tiles) / static_cast<double>(tiles);
    return static_cast<double>(wgs) * list * list < (d == 64 ? 3500.0 : 2000.0) * num_cus;
}

// Rows of a query tile (32 << shift) where `waves` waves of a workgroup may take them for several of the r heads of a KV head (emit_head_tiles).
int head_tile_shift(int r, int waves) { return r % waves == 0 ? 0 : r % (waves / 2) == 0 ? 1 : 2; }

// The eight-wave kernel (twice the heads per workgroup) may be taken for such a launch: prefill_pipe.hip has both sides' figures (tiles as above).  The padded launch goes
// by this alone; the packed one is held to longer lists by ahead_with_eight, which its rounds, at most half as many, cannot satisfy below 126 key tiles.
bool eight_waves(int64_t tiles, int64_t key_tiles, int Hq, int Hkv, int d) {
    return d == 128 && Hq / Hkv % 2 == 0 && tiles * Hq >= 512 && key_tiles >= 32 * tiles;
}

// Whether it is ahead on query tiles of several heads.  It runs in rounds of a workgroup per compute unit, with a first and a last turn that nothing covers
// (6 below, in halves of a key tile), and takes 3.5 % less for a key tile; of the four-wave workgroups two share a unit, one that is alone takes 0.7 of
// the time, and with fewer than eight heads to a KV head (four, two) their tiles have half the rows.  So what counts are the rounds and how long
// lists are.  Eight / four waves, us:
//   64/8 heads: 1 x 4096 behind 8192 1083 / 1119, 16 x 2048 behind 8000 0.979 of the time, 32 chunks behind up to 16384 (140 key tiles on average) 0.992, 8 x 4096
//   2023 / 1967, 32 x 1024 behind 2048 2436 / 2408, 4 x 300 behind 6000 (320 workgroups / 640) 295 / 255;
//   32/8: 2 x 1024 behind 8192 (256 / 512) 240 / 251, 16 chunks 2860 / 2798, 4 x 8192 1886 / 1860;  48/8: 4 x 300 behind 6000 (288 / 480) 295 / 175;
//   16/2: 2 x 1024 behind 8192 (128 / 256) 201 / 155, 1 x 4096 behind 8192 305 / 297.
// Over 120 launches of more than 32 key tiles a list this choice takes 0.4 % more than the faster one of the two; four
// waves everywhere 0.7 %, eight everywhere 3 %, and up to 70 %.  Over 90 launches in which it takes eight waves they are 1.8 % ahead of four, between 11 % ahead and 10 % behind (36 x 149 behind
// some 10000, 8/2 296 / 268; 16 x 128 behind some 9000, 32/8 316 / 286), and never behind 128 rows and two heads to a workgroup.
bool ahead_with_eight(const pk_plan& plan, int64_t tiles, int64_t key_tiles, int Hq, int Hkv, int num_cus) {
    const int r = Hq / Hkv;
    auto workgroups = [&](int waves) {
        const int shift = head_tile_shift(r, waves);
        int64_t n = 0;
        for (const int32_t q : plan.q_lens) n += (q + (32 << shift) - 1) >> (5 + shift);
        return n * Hkv * ((r << shift) / waves);
    };
    const int64_t four = workgroups(4), eight = workgroups(8), slots = 2 * num_cus, rest = four % slots;
    const double list = static_cast<double>(key_tiles) / static_cast<double>(tiles);
    double rounds4 = static_cast<double>(four) / num_cus, rounds8 = static_cast<double>(eight) / num_cus;
    if (four <= 16 * slots) {                      // (more rounds than that run into one another)
        rounds4 = 2.0 * static_cast<double>(four / slots) + (rest == 0 ? 0.0 : rest <= num_cus ? 1.4 : 2.0);
        rounds8 = std::ceil(rounds8);
    }
    return rounds8 * (1.93 * list + 6) < 0.985 * rounds4 * (list + 0.5);
}

// Writes the tiles in the given order (key-tile lists are re-based accordingly).
void emit_sched(const SchedBuild& sb, const std::vector<int32_t>& order, Builder& b, DeviceTables::PrefillSched& s) {
    std::vector<int32_t> desc, more_first, more, kv;
    desc.reserve(order.size() * kTileDescWords);
    more_first.reserve(order.size());
    kv.reserve(sb.kv.size());
    for (int32_t idx : order) {
        desc.push_back(static_cast<int32_t>(kv.size() / 2));
        desc.push_back(sb.n_kv[idx]);
        // per wave (8 bits each, saturating): how many key tiles at the START and at the END of the
        // list the wave skips (a packed query tile that straddles requests lists the key tiles of all
        // of them; the rows of one wave mostly belong to one)
        int32_t leading = 0, trailing = 0;
        for (int w = 0; w < 4; ++w) {
            auto code = [&](int32_t e) {
                return (sb.kv[2 * (static_cast<size_t>(sb.kv_first[idx]) + e) + 1] >> (8 + 2 * w)) & 3;
            };
            int32_t lead = 0, trail = 0;
            while (lead < sb.n_kv[idx] && lead < 255 && code(lead) == 0) ++lead;
            while (trail < sb.n_kv[idx] - lead && trail < 255 && code(sb.n_kv[idx] - 1 - trail) == 0) ++trail;
            leading |= lead << (8 * w);
            trailing |= trail << (8 * w);
        }
        desc.push_back(leading);
        desc.push_back(trailing);
        // The rows of a tile are runs of consecutive rows of one request each; most tiles are one
        // run, which sits in the descriptor itself (its Q row, lo, hi of tile row 0): the kernel
        // needs no second look-up before it can fetch its Q operand.  Further runs go to a list.
        const int32_t nr = sb.n_runs[idx];
        const int32_t* run = sb.runs.data() + 4 * static_cast<size_t>(sb.run_first[idx]);
        desc.push_back(sb.n_rows[idx] | (nr << 16));
        for (int x = 1; x < 4; ++x) desc.push_back(nr > 0 ? run[x] : 0);
        // words 8..10 and 11..13: first key rows and infos of the tile's first three key tiles (the last one
        // repeated if there are fewer), so that the kernel can request its first K/V tiles without waiting
        // for a look-up in the key-tile list
        for (int word = 0; word < 2; ++word)
            for (int e = 0; e < 3; ++e) {
                const int32_t ee = std::min(e, sb.n_kv[idx] - 1);
                desc.push_back(ee >= 0 ? sb.kv[2 * (static_cast<size_t>(sb.kv_first[idx]) + ee) + word] : 0);
            }
        desc.push_back(INT32_MAX); desc.push_back(0);
        more_first.push_back(static_cast<int32_t>(more.size() / 4));
        if (nr > 1) more.insert(more.end(), run + 4, run + 4 * static_cast<size_t>(nr));
        kv.insert(kv.end(), sb.kv.begin() + 2 * sb.kv_first[idx], sb.kv.begin() + 2 * (sb.kv_first[idx] + sb.n_kv[idx]));
    }
    s.n_tiles = s.n_query_tiles = static_cast<int32_t>(order.size());
    s.issued_pairs = sb.issued;
    s.tiles = b.add(desc);
    s.run_first = b.add(more_first); s.runs = b.add(more);
    s.kvtiles = b.add(kv);
}

// Launch order of query tiles: lists of more than half of the longest first, then of more than a quarter and so on, so that a launch ends with short
// ones; among those request by request, the one with the heaviest tile first, and inside a request the heaviest first:
// workgroups that run at the same time on one XCD then stream the same K/V rows, which keeps them in that XCD's L2.
// Request by request alone / in this order, us: 16 x 512 tokens, 32/8 heads 56.6 / 53.2, 16/8 35.2 / 31.9, 16/1 35.0 / 30.4, with d = 64 16/8
// 22.5 / 18.8, 8/8 13.6 / 12.5; 8 x 2048 16/8 144 / 133, 12/2 124 / 113, 16/1 146 / 134, d = 64 8/8 61.1 / 46.8; 24 x 1000 16/16
// 147.5 / 139.8; 28 x 560 64/8 231.6 / 228.0; long lists and many rounds of workgroups the same; 64 ragged prompts 347.7 / 351.1.  (Where ends_by_request says
// so, request by request alone.)
int halvings(int64_t list, int64_t longest) {
    int h = 0;
    while (list > 0 && list << (h + 1) <= longest) ++h;
    return h;
}
constexpr int kHalvings = 32;                      // (a list has less than 2^31 key tiles)

// Whether query tiles of one head stay request by request.  With one query head per KV head no workgroup but those of the request's other tiles reads a tile's K/V rows,
// and what the order above puts apart is read from memory again; all that it has to give is a shorter end.  So the one is weighed against the other, in launches of some
// rounds.  read_again: key tiles of the first tile of every further class of a request, ends_by: of the longest list among the last tiles that fill the
// chip, beyond those in the other order, both as parts of all (of what a slot goes through).  us, by the halvings of lists / request by request:
//   64 x 200, 16/16 heads 48.4 / 46.5;  32 x 512 32/32 151 / 132;  73 x 380 32/32 221 / 203;  28 of 139..478 32/32 66.0 / 60.3;  64 ragged prompts 32/32 408 / 394;  143 x 205
//   32/32 261 / 208;  99 x 178 behind up to 1278 32/32 489 / 372;  the other way 16 x 512 16/16 35.8 / 37.7, 24 x 1000 137.7 / 149.6, 3 x 1000 (0.7 rounds) 23.2 / 25.4.
// Over 577 such launches of 0.4 to 27 rounds this takes 0.6 % more than the faster order, up to 9 % (12 % once), the halvings 2.5 %, up to 32 %, request by request 1.7 %, up to 26 %.
// With head dimension 64 (half the bytes; 166 launches) the halvings take 0.3 % more than the faster order, 6 % at worst (64 x 200 16/16 27.7 / 25.8 us), request by request
// 5 %; with three, five and seven heads per KV head (199) 0.3 and 4.4 %.
bool stays_by_request(double rounds, double ends_by, double read_again, int r, int d) {
    return r == 1 && d == 128 && rounds > 2.5 && ends_by < 0.7 * read_again;
}

// With fewer than eight KV heads (one, two or four) neighbours in the launch order go to eight, four or two XCDs, and each reads the K/V rows of their request into its own
// L2.  So that four of them stay together, sets of four in a row are dealt over those XCDs, in one order and in the reverse one in turns: the tiles of a
// request come heaviest first, and with a fixed order the same XCD would get the heavier ones every time (8 x 4096 with 8/1 heads 244 -> 259 us).
// us before / now, 16 x 1024: 16/2 87.0 / 81.9, 8/1 46.8 / 42.6, 16/4 85.2 / 83.1, d = 64 16/2 48.4 / 45.6;  64 x 200 16/4 38.4 / 35.4, 16/2 35.2 / 33.3;  128 x 256 behind 7000 4/1
// 532 / 433, 8/1 855 / 818, 32/2 3220 / 3170;  8 x 4096 4/1 138 / 126, 8/1 253 / 241;  16 x 256 behind 4000 8/1 77.4 / 74.8;  16 chunks behind up to 16384 the same.  Over
// 96 shapes with one to four KV heads 1.7 % on average (sets of 2, 8 and 16: 1.2, 1.7, 1.2 %), 2.2 % slower at worst (64 ragged prompts 16/2 179.7 / 183.6).
struct DealOverXcds {
    int shift;                                     // 1 << shift sets to a block, one for each XCD of a KV head (0: tiles stay as they come)
    size_t whole;                                  // tiles in whole blocks
    DealOverXcds(size_t n, int Hkv) {
        shift = Hkv == 1 ? 3 : Hkv == 2 ? 2 : Hkv == 4 ? 1 : 0;
        whole = n >> (2 + shift) << (2 + shift);
    }
    size_t operator()(size_t x) const {            // where tile x in launch order goes
        if (shift == 0 || x >= whole) return x;
        const size_t block = x >> (2 + shift), sets = (size_t{1} << shift) - 1, set = x >> 2 & sets;
        return block << (2 + shift) | (x & 3) << shift | (block & 1 ? sets - set : set);
    }
};

// Query tiles of one request each and of 32 or 64 rows: the waves of a workgroup take its rows for several heads of a KV head (four waves: four
// heads or two), all on the same K/V tiles.  With 128 rows and one head a workgroup goes through the key tiles of all its rows while those of most
// waves are but a part of them: waves 0 and 1 do not see the last key tile of a causal tile, and where a tile holds several requests
// one wave or two work at a time.  (Rounds of a workgroup through a key tile, 128 rows / this: 64 ragged prompts 87000 / 77600, 44 chunks of
// 42 rows behind 320 with 64/8 heads 17700 / 7500, chunks of 512..2048 behind up to 16384 3.10 / 2.97 million.)  us, 128 rows / this:
//   64 ragged prompts, 32/8 heads 372.7 / 347.7;  44 x 42 behind 320, 64/8 66.5 / 44.7;  128 x 30, 32/8 28.5 / 18.6;  3 x 700 behind 600 51.2 / 42.6;
//   64 x 200, 64/8 153.8 / 131.9;  32 chunks of a 70B-shaped layer 10.61 / 10.33 ms;  8 x 2048, 64/8 544 / 537;  d = 64, 32/8:
//   256 x 64 behind 100 61.5 / 45.8;  64 x 200 39.7 / 34.3;  8 x 2048 159.0 / 159.1;  64 rows and two heads: 64 x 60, 16/8 12.3 / 10.2,
//   8 x 2048, 12/2 132 / 124, 40 x 200 behind 100 (a last tile of 8 rows) 16/8 34.0 / 34.9, 12/2 26.5 / 28.2.
// The key tiles of a request are a list that its query tiles share (a tile sees the first n of them and the keys up to `k_end`).
// A descriptor goes straight to its place in the launch order, which a count of the classes of lists gives: sorted as a list of tiles by those classes, and
// written entry by entry, the tables of many short prompts took twice as long as those of 128 rows and one head.  Host time of all tables, us, that way / this /
// 128 rows: 64 x 256 34.4 / 12.2 / 17.7, 512 x 16 59.6 / 24.8 / 28.7, 64 ragged prompts 83.7 / 20.3 / 51.4, chunks of a 70B-shaped layer 88 / 40 / 500.
void emit_head_tiles(const pk_plan& plan, const std::vector<int64_t>& q_start, const std::vector<int64_t>& kv_start, int Hkv, int row_shift,
                     Builder& b, DeviceTables::PrefillSched& s) {
    constexpr int BN = kPrefillBN;
    const int32_t rows = 32 << row_shift;
    // requests by the length of their list, the longest first, and by number among equals
    std::vector<uint64_t> requests(static_cast<size_t>(plan.n));
    size_t n_tiles = 0, n_entries = 0;
    for (int32_t rq = 0; rq < plan.n; ++rq) {
        const int32_t list = key_tiles_to(plan.kv_lens[rq]);
        requests[static_cast<size_t>(rq)] = static_cast<uint64_t>(INT32_MAX - list) << 32 | static_cast<uint32_t>(rq);
        n_tiles += static_cast<size_t>((plan.q_lens[rq] + rows - 1) / rows);
        n_entries += static_cast<size_t>(list);
    }
    std::sort(requests.begin(), requests.end());
    const int32_t longest = plan.n > 0 ? INT32_MAX - static_cast<int32_t>(requests[0] >> 32) : 0;
    // Where the tiles of each class of lists begin.  Inside a request lists get shorter tile by tile, and the class changes but a few times.
    auto each_tile = [&](int32_t rq, auto&& visit) {   // the heaviest tile first
        const int32_t lq = plan.q_lens[rq], ctx = plan.kv_lens[rq] - lq;
        int h = 0;
        for (int32_t t0 = (lq - 1) & -rows; t0 >= 0; t0 -= rows) {
            const int32_t n = std::min(rows, lq - t0), n_kv = key_tiles_to(ctx + t0 + n);
            while (static_cast<int64_t>(n_kv) << (h + 1) <= longest) ++h;
            visit(t0, n, n_kv, h);
        }
    };
    size_t next[kHalvings + 1] = {};
    for (const uint64_t key : requests)
        each_tile(static_cast<int32_t>(key & 0xFFFFFFFFu), [&](int32_t, int32_t, int32_t, int h) { ++next[h + 1]; });
    for (int h = 0; h < kHalvings; ++h) next[h + 1] += next[h];
    int32_t* desc = b.room(n_tiles * kTileDescWords, s.tiles);
    std::vector<int32_t> first_entry(static_cast<size_t>(plan.n));
    const DealOverXcds deal(n_tiles, Hkv);
    int64_t weight = 0;
    int32_t list = 0;
    for (const uint64_t key : requests) {
        const int32_t rq = static_cast<int32_t>(key & 0xFFFFFFFFu), kv = plan.kv_lens[rq];
        const int64_t ctx = kv - plan.q_lens[rq], ks0 = kv_start[rq];
        first_entry[static_cast<size_t>(rq)] = list;
        // (first key row, info) of the request's key tile e
        auto ks_of = [&](int32_t e) { return static_cast<int32_t>(ks0 + static_cast<int64_t>(e) * BN); };
        auto info_of = [&](int32_t e) { return static_cast<int32_t>(std::min<int64_t>(BN, kv - static_cast<int64_t>(e) * BN)) | 0xAA << 8; };
        each_tile(rq, [&](int32_t t0, int32_t n, int32_t n_kv, int h) {
            int32_t trailing = 0;
            for (int w = 0; w < 4; ++w) {
                const int32_t own = 32 * w >= n ? 0 : 32 * (w + 1) >= n ? n_kv : key_tiles_to(ctx + t0 + 32 * (w + 1));
                trailing |= std::min(n_kv - own, 255) << (8 * w);
                weight += own;
            }
            const int32_t e1 = std::min(1, n_kv - 1), e2 = std::min(2, n_kv - 1), hi = static_cast<int32_t>(ks0 + ctx + t0 + 1);
            const int32_t entry[kTileDescWords] = {list, n_kv, 0, trailing, n | 1 << 16, static_cast<int32_t>(q_start[rq] + t0), static_cast<int32_t>(ks0), hi,
                                                   ks_of(0), ks_of(e1), ks_of(e2), info_of(0), info_of(e1), info_of(e2), hi + n - 1, 0};
            std::copy(entry, entry + kTileDescWords, desc + deal(next[h]++) * kTileDescWords);
        });
        list += key_tiles_to(kv);
    }
    int32_t* entries = b.room(n_entries * 2, s.kvtiles);
    for (int32_t rq = 0; rq < plan.n; ++rq) {
        int32_t* e = entries + 2 * static_cast<size_t>(first_entry[static_cast<size_t>(rq)]);
        for (int64_t x = 0; x < plan.kv_lens[rq]; x += BN, e += 2) {
            e[0] = static_cast<int32_t>(kv_start[rq] + x);
            e[1] = static_cast<int32_t>(std::min<int64_t>(BN, plan.kv_lens[rq] - x)) | 0xAA << 8;
        }
    }
    s.row_shift = row_shift;
    s.n_tiles = static_cast<int32_t>(n_tiles);
    s.issued_pairs = weight * 32 * BN;
}

// Launches whose time is that of a few workgroups with long lists (a chunk or a handful of rows behind a long context, few heads): the lists are cut into
// pieces of (nearly) the same length, a workgroup each, and a second launch puts the pieces together (prefill_merge).  A key tile takes a workgroup 0.87 us
// whether it has a compute unit to itself or shares it, so that a launch takes as long as its longest list or, if that is more, as all lists dealt over the units; pieces cost
// a launch, a start each, and 17 KiB per 32 rows and head (9 with d = 64) that are written and read.  us, whole lists / pieces of the length that ListSplit
// finds best, d = 128: 1 x 64 rows behind 8000 with 8/8 heads (8 workgroups of 126 key tiles) 113 / 21; 32/8 heads 1 x 16 behind 16000 217 / 28, behind 2000 30.7 / 14.9,
// 1 x 128 behind 8192 127 / 30, 1 x 512 behind 8192 134 / 83, 4 x 100 behind 3000 52.0 / 38.5; 4/1 heads 8 of 68..112 behind up to 4600 71 / 21, 1 x 4096 64.7 / 35.3;
// 8/2 heads 1 x 1105 20.6 / 19.0; d = 64: 1 x 64 behind 8000 with 8/8 88.8 / 17.7.  Of 800 launches (1 to 40 requests, up to 20000 keys, eleven head
// shapes) 173 get pieces, twice as fast on average; one of them lost (1 x 1124 with 12/2 heads 21.1 / 21.7).
struct ListSplit {
    int d, num_cus;
    double tile() const { return d == 64 ? 0.66 : 0.87; }          // us
    // workgroups, their key tiles and the longest list
    double run(double wgs, double total, int32_t longest) const {
        const double per_cu = wgs / num_cus, rounds = per_cu <= 1 ? 1.0 : (per_cu + std::ceil(per_cu)) / 2;   // (one more on some units than on others)
        return 6.0 + 1.5 * (rounds - 1) + tile() * std::max<double>(longest, rounds * total / wgs * (d == 64 && rounds > 1 ? 0.8 : 1.0));
    }
    double merge(double pieces, double most) const { return 5.0 + 0.3 * most + pieces * (d == 64 ? 0.008 : 0.012); }
};
void split_lists(const pk_plan& plan, const std::vector<int64_t>& q_start, const std::vector<int64_t>& kv_start, int Hq, int head_shift, int num_cus, Builder& b,
                 DeviceTables& t) {
    constexpr int32_t SHORTEST = 13;               // key tiles: the second launch takes as long as six
    DeviceTables::PrefillSched& s = t.packed;
    const int32_t* desc0 = b.host.data() + s.tiles.offset / sizeof(int32_t);
    const int64_t units0 = static_cast<int64_t>(t.Hkv) * ((Hq / t.Hkv << s.row_shift) / 4);        // workgroups of a query tile
    int32_t longest = 0;
    int64_t total = 0;
    for (int32_t x = 0; x < s.n_tiles; ++x) {
        longest = std::max(longest, desc0[kTileDescWords * x + 1]);
        total += desc0[kTileDescWords * x + 1];
    }
    if (longest < SHORTEST) return;
    const ListSplit est{t.d, num_cus};
    const double whole = est.run(static_cast<double>(s.n_tiles * units0), static_cast<double>(total * units0), longest);
    double best = 0.92 * whole;
    if (est.run(num_cus, static_cast<double>(total * units0), 0) + est.merge(0, 2) >= best) return;       // (all units busy from the first to the last)
    // the pieces are of tiles of several heads where there are such: none of their waves is idle but for a request's last rows
    const int64_t units = static_cast<int64_t>(t.Hkv) * ((Hq / t.Hkv << head_shift) / 4);
    const int32_t rows = 32 << head_shift;
    std::vector<int32_t> lists;
    for (int32_t i = 0; i < plan.n; ++i)
        for (int32_t t0 = 0, lq = plan.q_lens[i]; t0 < lq; t0 += rows) lists.push_back(key_tiles_to(plan.kv_lens[i] - lq + std::min(lq, t0 + rows)));
    total = std::accumulate(lists.begin(), lists.end(), int64_t{0});
    int32_t most = 0;
    for (int32_t len = 4; len < longest; len += std::max(1, len / 4)) {
        int64_t n = 0, pieces = 0;
        int32_t parts = 1, piece = 0;
        for (const int32_t l : lists) {
            const int32_t p = (l + len - 1) / len;
            n += p;
            pieces += p > 1 ? p : 0;
            parts = std::max(parts, p);
            piece = std::max(piece, (l + p - 1) / p);
        }
        const double time = est.run(static_cast<double>(n * units), static_cast<double>(total * units), piece) + est.merge(static_cast<double>(pieces * units), parts);
        if (time < best) { best = time; most = len; }
    }
    if (most == 0) return;
    std::vector<int32_t> host;
    Builder own(host);
    DeviceTables::PrefillSched h = s;
    const bool other = head_shift != s.row_shift;
    if (other) emit_head_tiles(plan, q_start, kv_start, t.Hkv, head_shift, own, h);
    const int32_t* tables = (other ? host : b.host).data();
    const int32_t *desc = tables + h.tiles.offset / sizeof(int32_t), *kv = tables + h.kvtiles.offset / sizeof(int32_t);
    std::vector<int32_t> pieces, merges;
    int32_t slots = 0;
    for (int32_t x = 0; x < h.n_tiles; ++x, desc += kTileDescWords) {
        const int32_t n_kv = desc[1], n = std::max(1, (n_kv + most - 1) / most);
        if (n > 1) {
            const int32_t entry[4] = {slots, n, desc[5], desc[4] & 0xFFFF};
            merges.insert(merges.end(), entry, entry + 4);
        }
        for (int32_t p = 0; p < n; ++p) {
            const int32_t e0 = static_cast<int32_t>(static_cast<int64_t>(n_kv) * p / n), e1 = static_cast<int32_t>(static_cast<int64_t>(n_kv) * (p + 1) / n);
            int32_t piece[kTileDescWords];
            std::copy(desc, desc + kTileDescWords, piece);
            piece[0] = desc[0] + e0;
            piece[1] = e1 - e0;
            piece[2] = piece[3] = 0;
            for (int w = 0; w < 4; ++w) {          // where this wave's key tiles begin and end
                const int32_t lead = desc[2] >> (8 * w) & 0xFF, trail = desc[3] >> (8 * w) & 0xFF;
                piece[2] |= std::min(255, std::max(0, std::min(lead, e1) - e0)) << (8 * w);
                piece[3] |= std::min(255, std::max(0, e1 - std::max(n_kv - trail, e0))) << (8 * w);
            }
            for (int32_t e = 0; e < 3; ++e)
                for (int word = 0; word < 2; ++word) {
                    const size_t at = 2 * (static_cast<size_t>(desc[0]) + std::max(0, std::min(e0 + e, e1 - 1)));
                    piece[8 + 3 * word + e] = n_kv > 0 ? kv[at + word] : 0;
                }
            piece[15] = n > 1 ? ++slots : 0;
            pieces.insert(pieces.end(), piece, piece + kTileDescWords);
        }
    }
    if (merges.empty()) return;
    s.n_pieces = static_cast<int32_t>(pieces.size() / kTileDescWords);
    s.n_merges = static_cast<int32_t>(merges.size() / 4);
    s.piece_shift = head_shift;
    s.piece_kvtiles = other ? b.add(std::vector<int32_t>(kv, kv + h.kvtiles.count)) : s.kvtiles;
    s.pieces = b.add(pieces);
    s.merges = b.add(merges);
    s.whole_us = whole;
    t.prefill_part_bytes = static_cast<size_t>(slots) * units * 4 * 64 * (2 * t.d + 16);
}

// packed: tiles over each group's packed row stream, heaviest tile first
void build_prefill_packed(const pk_plan& plan, const std::vector<int64_t>& q_start,
                          const std::vector<int64_t>& kv_start, int Hq, int num_cus, Builder& b, DeviceTables& t) {
    constexpr int BM = kPrefillBM;
    // A batch so small that even one tile per request piece leaves workgroup slots empty (two per
    // compute unit) gains nothing from sharing tiles between requests: a shared tile walks the key
    // tiles of both requests one after the other, which only lengthens the longest workgroup.
    int64_t aligned_tiles = 0;
    for (int32_t i = 0; i < plan.n; ++i) aligned_tiles += (plan.q_lens[i] + BM - 1) / BM;
    const bool may_share = aligned_tiles * Hq > 2 * static_cast<int64_t>(num_cus);
    // A request that does not fit into what is left of the current tile shares it only if
    // that saves the request a tile of its own (its head then rides along with few key
    // tiles); otherwise the tile is closed and the request starts on a fresh one: a shared
    // tile walks the key tiles of both requests one after the other and runs them masked.
    auto starts_fresh = [&](int32_t filled, int32_t lq) {
        return filled > 0 && (!may_share || BM - filled < (lq - 1) % BM + 1);      // (rows of its last tile when it starts fresh)
    };
    // What the choice of the kernel goes by: the tiles and their key tiles (a full tile has two more of them than the one before it).
    int64_t n_tiles = 0, key_tiles = 0, total_rows = 0;
    for (const Group& g : plan.groups) {
        int32_t filled = 0;                        // rows of the tile that is open
        for (const Member& m : g.members) {
            const int32_t lq = plan.q_lens[m.req];
            const int64_t ctx = plan.kv_lens[m.req] - lq;
            if (starts_fresh(filled, lq)) { ++n_tiles; filled = 0; }
            const int32_t head = std::min(BM - filled, lq);
            key_tiles += key_tiles_to(ctx + head);
            total_rows += lq;
            filled += head;
            if (filled < BM) continue;
            const int32_t full = (lq - head) / BM, rest = lq - head - full * BM;
            key_tiles += full * static_cast<int64_t>(key_tiles_to(ctx + head + BM)) + static_cast<int64_t>(full) * (full - 1) + (rest > 0 ? key_tiles_to(ctx + lq) : 0);
            n_tiles += 1 + full;
            filled = rest;
        }
        if (filled > 0) ++n_tiles;
    }
    DeviceTables::PrefillSched& s = t.packed;
    s.light = light_launch(n_tiles, key_tiles, Hq, t.d, num_cus);
    s.eight = !s.light && eight_waves(n_tiles, key_tiles, Hq, t.Hkv, t.d) && ahead_with_eight(plan, n_tiles, key_tiles, Hq, t.Hkv, num_cus);
    const int row_shift = head_tile_shift(Hq / t.Hkv, s.eight ? 8 : 4);
    // Where every tile of 128 rows and head has a compute unit of its own, and waves of the tile with the longest list (at least one) or a fifth of all rows are empty, fewer
    // waves share a unit's LDS with those tiles than with several heads to a workgroup.  128 rows / several heads, us: 1 x 64 behind 8000 with 16 heads 113 / 121, d = 64 89 / 97; 7 x 57 behind
    // 2500 with 16 heads 40.0 / 42.5, 32 heads 40.4 / 42.6, 64 heads (448 workgroups) 58.3 / 45.9; 3 x 200 behind 300 with 32 heads 12.6 / 13.1, 64 heads (384) 18.6 / 19.0; 2 of 382
    // and 407, 8/2 10.6 / 11.2; 4 of 315..554, 8/2 12.7 / 13.5; 2 x 440, 16/8 and d = 64 8.5 / 9.0; 6 x 211 behind up to 1161, 8/1 25.2 / 25.9; with a full tile the other way: 1 x 1000
    // 16/2 20.2 / 19.8, 2 x 128 behind 4000 66.3 / 65.3, 5 of 173..358 (last tile 102 rows) 8/4 10.6 / 10.4.
    bool spread = plan.n > 0 && aligned_tiles * Hq <= num_cus;
    if (spread) {
        const int32_t rq = static_cast<int32_t>(std::max_element(plan.kv_lens.begin(), plan.kv_lens.end()) - plan.kv_lens.begin());
        spread = (plan.q_lens[rq] - 1) % BM < BM - 32 || 5 * total_rows <= 4 * BM * aligned_tiles;
    }
    if (!plan.decode_only && t.dtype == PK_BF16 && row_shift < 2 && !spread) {
        emit_head_tiles(plan, q_start, kv_start, t.Hkv, row_shift, b, s);
        s.n_query_tiles = static_cast<int32_t>(n_tiles);
        if (s.light) split_lists(plan, q_start, kv_start, Hq, row_shift, num_cus, b, t);
        return;
    }
    SchedBuild sb;
    sb.reserve(static_cast<size_t>(n_tiles), static_cast<size_t>(plan.n + n_tiles), static_cast<size_t>(key_tiles));
    std::vector<RowRun> runs;                      // of the tile that is open
    std::vector<int32_t> tile_req;                 // request of a tile's first row
    tile_req.reserve(static_cast<size_t>(n_tiles));
    int32_t filled = 0;                            // rows of the tile that is open
    auto close_tile = [&] {
        tile_req.push_back(runs[0].req);
        add_tile(plan, q_start, kv_start, runs.data(), runs.data() + runs.size(), false, sb);
        runs.clear();
        filled = 0;
    };
    for (const Group& g : plan.groups) {
        for (const Member& m : g.members) {
            const int32_t lq = plan.q_lens[m.req];
            if (starts_fresh(filled, lq)) close_tile();
            for (int32_t x = 0; x < lq;) {
                const int32_t take = std::min(BM - filled, lq - x);
                runs.push_back({filled, take, m.req, x});
                filled += take;
                x += take;
                if (filled == BM) close_tile();
            }
        }
        if (filled > 0) close_tile();
    }
    std::vector<int32_t> order(sb.n_kv.size());
    std::iota(order.begin(), order.end(), 0);
    std::vector<int64_t> req_weight(static_cast<size_t>(plan.n), 0);
    for (size_t x = 0; x < tile_req.size(); ++x)
        req_weight[static_cast<size_t>(tile_req[x])] = std::max(req_weight[static_cast<size_t>(tile_req[x])], sb.weight[x]);
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
        const int32_t rx = tile_req[static_cast<size_t>(x)], ry = tile_req[static_cast<size_t>(y)];
        if (rx != ry) {
            if (req_weight[static_cast<size_t>(rx)] != req_weight[static_cast<size_t>(ry)])
                return req_weight[static_cast<size_t>(rx)] > req_weight[static_cast<size_t>(ry)];
            return rx < ry;
        }
        return sb.weight[x] > sb.weight[y];
    });
    const int32_t longest = sb.n_kv.empty() ? 0 : *std::max_element(sb.n_kv.begin(), sb.n_kv.end());
    size_t next[kHalvings + 1] = {};
    for (const int32_t x : order) ++next[halvings(sb.n_kv[x], longest) + 1];
    for (int h = 0; h < kHalvings; ++h) next[h + 1] += next[h];
    const std::vector<int32_t> by_request(order);
    double read_again = 0;
    int32_t before = -1;                           // the tile before, and its class
    int before_h = 0;
    for (const int32_t x : by_request) {
        const int h = halvings(sb.n_kv[x], longest);
        if (before >= 0 && tile_req[static_cast<size_t>(x)] == tile_req[static_cast<size_t>(before)] && h != before_h) read_again += sb.n_kv[x];
        order[next[h]++] = before = x;
        before_h = h;
    }
    const int slots = 2 * num_cus;                 // workgroups at a time
    auto end_of = [&](const std::vector<int32_t>& o) {
        const size_t last = std::min(o.size(), static_cast<size_t>(std::max(1, slots / Hq)));
        int32_t list = 0;
        for (size_t x = o.size() - last; x < o.size(); ++x) list = std::max(list, sb.n_kv[o[x]]);
        return list;
    };
    const double rounds = static_cast<double>(n_tiles) * Hq / slots, work = std::max(1.0, static_cast<double>(key_tiles));
    // (with a compute unit for each of them all workgroups start at once, and no order ends earlier: 461, 852 and 403 rows with 16/2 heads 18.3 by halvings, 17.9 by request)
    if (n_tiles * Hq <= num_cus || stays_by_request(rounds, (end_of(by_request) - end_of(order)) * slots / (work * Hq), read_again / work, Hq / t.Hkv, t.d)) order = by_request;
    emit_sched(sb, order, b, s);
    if (!plan.decode_only && t.dtype == PK_BF16 && s.light && !may_share) split_lists(plan, q_start, kv_start, Hq, row_shift, num_cus, b, t);
}

}  // namespace

// packed, of a decode plan: hardly ever asked for, so it is built on first use into its own host image (uploaded behind the partial results).  Building the
// tables of 48 / 400 decode requests took 11.4 / 36.5 us of the host with it among them, and takes 4.3 / 15.4 without.
void build_prefill_of_decode(const pk_plan& plan, DeviceTables& t) {
    std::vector<int64_t> q_start(static_cast<size_t>(plan.n) + 1, 0), kv_start(static_cast<size_t>(plan.n) + 1, 0);
    for (int32_t i = 0; i < plan.n; ++i) {
        q_start[i + 1] = q_start[i] + plan.q_lens[i];
        kv_start[i + 1] = kv_start[i] + plan.kv_lens[i];
    }
    t.host_packed.clear();
    t.packed = DeviceTables::PrefillSched();
    Builder b(t.host_packed);
    build_prefill_packed(plan, q_start, kv_start, t.Hq, t.num_cus, b, t);
    t.host_packed.resize((t.host_packed.size() + 63) / 64 * 64, 0);
    t.packed_built = true;
}

// padded: request-aligned grid (request, tile) sized by the longest request, natural order.
// Built on first use into its own host image (uploaded behind the partial results).
void build_prefill_padded(const pk_plan& plan, DeviceTables& t) {
    constexpr int BM = kPrefillBM;
    std::vector<int64_t> q_start(static_cast<size_t>(plan.n) + 1, 0), kv_start(static_cast<size_t>(plan.n) + 1, 0);
    for (int32_t i = 0; i < plan.n; ++i) {
        q_start[i + 1] = q_start[i] + plan.q_lens[i];
        kv_start[i + 1] = kv_start[i] + plan.kv_lens[i];
    }
    int32_t max_tiles = 0;
    for (int32_t i = 0; i < plan.n; ++i) max_tiles = std::max(max_tiles, (plan.q_lens[i] + BM - 1) / BM);
    SchedBuild sb;
    for (int32_t i = 0; i < plan.n; ++i) {
        for (int32_t tt = 0; tt < max_tiles; ++tt) {
            const int32_t rows = std::min(plan.q_lens[i] - tt * BM, BM);
            const RowRun run = {0, rows, i, tt * BM};
            if (rows <= 0) add_idle_tile(sb);
            else add_tile(plan, q_start, kv_start, &run, &run + 1, true, sb);
        }
    }
    std::vector<int32_t> order(sb.n_kv.size());
    std::iota(order.begin(), order.end(), 0);
    t.host_padded.clear();
    Builder b(t.host_padded);
    emit_sched(sb, order, b, t.padded);
    const int64_t key_tiles = std::accumulate(sb.n_kv.begin(), sb.n_kv.end(), int64_t{0});
    t.padded.light = light_launch(t.padded.n_tiles - std::count(sb.n_kv.begin(), sb.n_kv.end(), 0), key_tiles, t.Hq, t.d, t.num_cus);
    t.padded.eight = !t.padded.light && eight_waves(t.padded.n_tiles, key_tiles, t.Hq, t.Hkv, t.d);
    t.host_padded.resize((t.host_padded.size() + 63) / 64 * 64, 0);
    t.padded_built = true;
}

namespace {

// Upper bound (bytes) of the padded schedule's tables, without building them.
size_t padded_bound_bytes(const pk_plan& plan) {
    constexpr int64_t BM = kPrefillBM, BN = kPrefillBN;
    int64_t max_tiles = 0, kv_entries = 0;
    for (int32_t i = 0; i < plan.n; ++i) max_tiles = std::max<int64_t>(max_tiles, (plan.q_lens[i] + BM - 1) / BM);
    for (int32_t i = 0; i < plan.n; ++i) {
        const int64_t ctx = plan.kv_lens[i] - plan.q_lens[i];
        for (int64_t tt = 0; tt * BM < plan.q_lens[i]; ++tt)
            kv_entries += (ctx + std::min<int64_t>(plan.q_lens[i], (tt + 1) * BM) + BN - 1) / BN;
    }
    const int64_t tiles = max_tiles * plan.n;
    const int64_t ints = tiles * kTileDescWords + tiles + 2 * kv_entries + 6 * 64;   // a padded tile is one run: the run list is empty
    return static_cast<size_t>((ints + 63) / 64 * 64) * sizeof(int32_t);
}

// Bytes of the packed prefill schedule of a decode plan, without building it: a tile is closed before a row that does not fit into what is left of it, so that
// every request is one run of one row, and all its key tiles are listed once.
size_t packed_bytes_of_decode(const pk_plan& plan, int Hq, int num_cus) {
    constexpr int64_t BM = kPrefillBM;
    const bool may_share = static_cast<int64_t>(plan.n) * Hq > 2 * static_cast<int64_t>(num_cus);
    int64_t tiles = 0, key_tiles = 0;
    for (const Group& g : plan.groups) {
        const int64_t rows = static_cast<int64_t>(g.members.size());
        tiles += may_share ? (rows + BM - 1) / BM : rows;
    }
    for (const int32_t kv : plan.kv_lens) key_tiles += key_tiles_to(kv);
    auto aligned = [](int64_t ints) { return (ints + 63) / 64 * 64; };
    return static_cast<size_t>(aligned(tiles * kTileDescWords) + aligned(tiles) + aligned(4 * (plan.n - tiles)) + aligned(2 * key_tiles)) * sizeof(int32_t);
}

}  // namespace

size_t kv_buf_bytes(const pk_plan& plan, int Hkv, int d, int dtype) {
    const size_t elem = dtype == PK_F32 ? 4 : 2;
    return static_cast<size_t>(plan.buf_tokens) * Hkv * d * 2 * elem;
}

namespace {
void fill_tables(const pk_plan& plan, int Hq, int Hkv, int d, int dtype, int num_cus, bool may_choose, DeviceTables& t) {
    t = DeviceTables();
    t.Hq = Hq; t.Hkv = Hkv; t.d = d; t.dtype = dtype;
    t.num_cus = num_cus;
    Builder b(t.host);
    // (room for most plans: grown table by table the image was copied, and its fresh pages touched, several times)
    t.host.reserve(static_cast<size_t>(plan.n) * (plan.decode_only ? 40 + (may_choose ? Hkv : 0) : 24) + static_cast<size_t>(plan.buf_tokens / kDecodeBlock) + 16 * 64);
    std::vector<int64_t> q_start(static_cast<size_t>(plan.n) + 1, 0), kv_start(static_cast<size_t>(plan.n) + 1, 0);
    for (int32_t i = 0; i < plan.n; ++i) {
        q_start[i + 1] = q_start[i] + plan.q_lens[i];
        kv_start[i + 1] = kv_start[i] + plan.kv_lens[i];
    }
    t.q_start = b.add(std::vector<int32_t>(q_start.begin(), q_start.end()));
    t.kv_start = b.add(std::vector<int32_t>(kv_start.begin(), kv_start.end()));
    build_reorg(plan, b, t);
    size_t packed_bytes = 0;                       // of tables that are built later
    if (plan.decode_only) {
        build_decode(plan, Hq, Hkv, d, dtype, num_cus, may_choose, b, t);
        packed_bytes = packed_bytes_of_decode(plan, Hq, num_cus);
    } else {
        build_prefill_packed(plan, q_start, kv_start, Hq, num_cus, b, t);
        t.packed_built = true;
    }
    t.host.resize((t.host.size() + 63) / 64 * 64, 0);
    t.tables_bytes = t.host.size() * sizeof(int32_t);
    t.partial_offset = t.tables_bytes;
    t.partial_bytes = static_cast<size_t>(t.dec.n_parts) * Hq * (static_cast<size_t>(d) + 1) * sizeof(float) + t.prefill_part_bytes;   // (no plan has both)
    t.decode_only_bytes = t.partial_offset + t.partial_bytes + packed_bytes;       // (whether a plan fits the fixed scratch counts all its tables)
    if (t.dec.chosen) {
        // what the plan would need with a wave per item and one split decides whether it may use the fixed scratch
        auto aligned = [](size_t words) { return (words + 63) / 64 * 64; };
        auto words = [&](int32_t items, int32_t members) { return aligned(8 * static_cast<size_t>(items)) + 2 * aligned(static_cast<size_t>(members)); };     // with their slots
        const size_t by_waves = t.tables_bytes + packed_bytes + sizeof(int32_t) * (words(t.dec.wave_items, t.dec.wave_members) -
            words(t.dec.n_items, t.dec.n_members) - (t.dec.group ? aligned(static_cast<size_t>(plan.n) * Hkv) : 0)) +
            static_cast<size_t>(t.dec.wave_parts) * Hq * (static_cast<size_t>(d) + 1) * sizeof(float);
        t.group_over_scratch = t.decode_only_bytes > PK_STATIC_SCRATCH_BYTES && by_waves <= PK_STATIC_SCRATCH_BYTES;
        t.decode_only_bytes = by_waves;
    }
    if (plan.decode_only) {
        // the padded comparison kernel keeps (request, split) partials in the same region: the
        // same number of splits for every request, sized by the longest -- at most 64, each a
        // multiple of 32 tokens and at least 512 tokens long (enough waves to fill the chip from the
        // long requests alone; more splits only add empty grid slots and partial results)
        int32_t max_len = 0;
        for (int32_t L : plan.kv_lens) max_len = std::max(max_len, L);
        int32_t split = std::max(512, ((max_len + 63) / 64 + 31) / 32 * 32);
        t.pad_split_tokens = split;
        t.pad_n_splits = (max_len + split - 1) / split;
        const size_t pad_bytes = static_cast<size_t>(plan.n) * t.pad_n_splits * Hq * (static_cast<size_t>(d) + 1) * sizeof(float);
        t.partial_bytes = std::max(t.partial_bytes, pad_bytes);
    }
    t.packed_offset = (t.partial_offset + t.partial_bytes + 255) / 256 * 256;
    t.padded_offset = (t.packed_offset + packed_bytes + 255) / 256 * 256;
    t.total_bytes = (t.padded_offset + padded_bound_bytes(plan) + 255) / 256 * 256;
}
}  // namespace

void build_tables(const pk_plan& plan, int Hq, int Hkv, int d, int dtype, int num_cus, DeviceTables& t) {
    // (what may not be chosen in the second: workgroups for items, and a split for shared segments)
    fill_tables(plan, Hq, Hkv, d, dtype, num_cus, true, t);
    if (t.group_over_scratch) fill_tables(plan, Hq, Hkv, d, dtype, num_cus, false, t);
}

}  // namespace pk

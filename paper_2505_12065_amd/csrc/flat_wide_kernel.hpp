// Exact (flat) retrieval on the matrix cores (Section 2.1 of the paper: exact retrieval; the batch stands for the
// agent's concurrent requests).  The score matrix S = X Q^T is a dense contraction:
//
//   workgroup tile  32 WMF NWM corpus rows x 32 WNF NWN queries, NWM x NWN wavefronts
//   wavefront tile  32 WMF rows x 32 WNF queries = WMF x WNF MFMA 32x32x16 accumulators
//   K loop          stages of 64 bytes of a row (the two large tiles) or 128 (the others), 2 to 4 of them in LDS; every stage is
//                   filled by direct global->LDS loads issued one to three stages ahead.  One load instruction brings a 1 KB
//                   block, 16 rows x 64 B or 8 rows x 128 B (whole cache lines); inside a row the 16-byte chunks sit in slots
//                   XOR-swizzled by the row number, so the MFMA operand reads (32 rows x one chunk) hit all banks
//   epilogue        the largest score of every group of 1, 4, 16, 32 or 16 WMF rows (all of one lane's), nothing else:
//                   maxima[q, group].  flat_pick_kernel finds the k best groups of a query, which hold its k best
//                   rows, scores their rows once more by the same instructions and picks the rows
//
// A workgroup walks a slab of corpus tiles for one query tile.  Blocks are numbered so that neighbours, which run on one
// XCD, share the operand that is read more often: the slab where the corpus is the larger, else the query tile
// (977 x 768, B = 5000: 26 -> 23 us with the stores below; every XCD had read all the queries).
//
// Stages of whole lines halve the barriers and the L2's requests; three of them leave room for tiles of 256 x 128 at most.
// 300 k x 768, B = 128: 132 us by 512 x 128 tiles of half lines, 112 by 256 x 128 of whole ones; 123 457 x 776, B = 77 (a row of
// 12 1/8 lines) 70 -> 64.  With whole lines a 64 x 64 tile spends 810 clocks a stage, 150 of them on products: its
// loads are there, barrier, addresses and LDS reads follow each other.  So the steps inside a tile run in a loop without a look
// at where the loads are, and the addresses are made while the reads run: 977 x 768, B = 5000 32.2 -> 31.2 us a search, 16 k x 768,
// B = 256 24.1 -> 23.6, 1024 x 768, B = 512 11.9 -> 11.6 (the large tiles, two waves of them on a SIMD, lose 4 % that way: 1 M x
// 768, B = 512 895 -> 937; reading the operands a stage ahead gains nothing at any).
//
// BY_LINE: rows that are no whole number of lines.  128 bytes of such a row lie in two lines, each of which the L2 serves twice (1 M x 776,
// B = 128: 37 M requests, 21 M for x 768 and x 832), so stages go by the lines of memory instead: a row's first chunk is chunk `lead` of its first
// line.  A line's chunks go to the LDS places of their number in the row modulo 8, so operand reads stay what they are, and the products of a
// step, one line later, take a lane's chunks from the line before where that had them: same operands, same bits.  Only corpus rows go
// by lines; with the queries too, both lines' operands and the choice between them take 256 registers and twice the selects (160 k x 776, B = 77 57.2 ->
// 61.5 us from the caches, this 57.5 -> 57.2).  us, stages of rows / of lines: 1 M x 776, B = 128 412 / 367; 123 457 x 776, B = 77
// 56.4 / 51.3; 300 k x 264, B = 40 51.2 / 45.9; 800 k x 864, B = 77 315 / 297.
//
// The epilogue is what decides at most sizes.  Sorted lists per lane, with thresholds from a sampling pass, cost two to
// three launches, 130 registers of lists and queues, and insertions that never become rare unless a slab has
// thousands of rows: 3 to 10 times the products' time below 200 k rows.  Maxima take a few instructions per
// tile, no threshold and no warm-up, so short slabs and small tiles are as good as long ones.
#pragma once

#include "common.hpp"
#include "launch.hpp"

namespace ann {

#define ANN_GLOBAL_TO_LDS_16(gptr, lptr)                                                          \
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gptr),      \
                                     (__attribute__((address_space(3))) void *)(lptr), 16, 0, 0)

// wait until at most `n` of this wave's vector-memory operations are outstanding
template <int n>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(n >= 0 && n < 64, "vmcnt is a 6-bit field");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (n & 15) | ((n >> 4) << 14));
}

// a barrier that waits for no memory operation
__device__ __forceinline__ void bare_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// ... and that a wave comes to with its LDS reads in registers
__device__ __forceinline__ void barrier_after_reads() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

static __device__ __align__(16) unsigned char zero_row_end[16];          // what lies behind the end of a row

// X [N, d], Q [B, d] 16-bit, d a multiple of 8.  maxima [B, n]: n = groups of all tiles, in the order of wide_row.
// gridDim.x = P * NT; the tiles are dealt to P slabs.
// 2^gs_log: rows per group, ONE: 1, else 4, 16, 32 or 16 WMF (two kernels: the stores of single rows are 40 % of the code,
// and in one kernel with the rest they cost 1 M x 768, B = 512 1 %).  Rows that do not exist or do not come after a query's boundary count as NaN.
template <class T, class C, bool ONE, bool BY_LINE>
__global__ __launch_bounds__(C::THREADS, C::PER_CU * C::WAVES / 4) void flat_wide_kernel(
    const void *__restrict__ X, int64_t N, int d, const void *__restrict__ Q, int B, float *__restrict__ maxima, int64_t n,
    int P, int NT, int gs_log, After after) {
    constexpr int WMF = C::WMF, WNF = C::WNF, NST = C::STAGES, LPW = C::LPW, BM = C::BM;
    constexpr int SB = C::SB, CPR = C::CPR, RPB = C::RPB, NKH = SB / 32;
    extern __shared__ __align__(16) unsigned char stage_mem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % C::NWM, wn = wave / C::NWM;
    const int l32 = lane & 31, lhi = lane >> 5;
    const int rb = d * 2, ksteps = (rb + SB - 1) / SB;
    static_assert(!BY_LINE || SB == 128, "a stage is a line");
    const int nch = rb >> 4;
    auto lead = [&](int64_t row) { return (int)((reinterpret_cast<uintptr_t>(X) >> 4) + (uint64_t)row * nch) & 7; };
    // stages of a tile; leads are multiples of `common`, so 8 - common is the longest
    const uint32_t common = (uint32_t)nch | 8u | (uint32_t)(reinterpret_cast<uintptr_t>(X) >> 4);
    const int lines = BY_LINE ? (nch + 8 - (int)(common & -common) + 7) >> 3 : ksteps;

    const int lb = xcd_block();
    const bool by_query = N < B;
    const int nt = by_query ? lb / P : lb % NT, slab = by_query ? lb % P : lb / NT, n0 = nt * C::BN;
    const int64_t mtiles = (N + BM - 1) / BM;
    const int64_t t0 = mtiles * slab / P, t1 = mtiles * (slab + 1) / P;
    const int total = (int)(t1 - t0) * lines;

    // Block e of a stage: blocks 0 .. A_BLK - 1 corpus rows, the rest queries.  Lane l fetches row l / CPR of the block;
    // LDS slot l % CPR of that row receives chunk (l % CPR) ^ swz(row) of the stage's bytes of the row: 16 rows, which an operand
    // read takes at a time, lie in 16 different places of the 256 bytes that
    // the banks hold (whole lines swizzled by the row's lowest bits: half of the reads' clocks were conflicts, 977 x 768, B = 5000 31.1
    // -> 30.4 us).
    auto swz = [](int row) { return SB == 64 ? (row >> 2) & 3 : (row >> 1) & 7; };
    auto my_chunk = [&](int e) { return (lane & (CPR - 1)) ^ swz((wave * LPW + e) * RPB + lane / CPR); };
    // Address of a load = uniform base (corpus: start of the tile, advanced per k step; queries: start of the query
    // tile) + a 32-bit per-lane offset that does not change from tile to tile, except in the ragged last tile
    // where rows are clamped to N - 1.  In the last stage of rows that end inside it, chunks behind the end come
    // from a row of zeros.
    // (Lambdas of the K loop are inlined by order: those of the 128 x 128 tile were called otherwise, its accumulators in scratch memory, 121 us
    // instead of 25 at 977 x 768, B = 5000.  The other tiles' code is the same either way.)
    // BY_LINE: the offset in the row's first line may lie before the row, and so before the tile.
    uint32_t loff[LPW], first_chunk = 0;                  // first_chunk: 7 more than the chunk of its row that the lane brings first, 4 bits each
    static_assert(LPW <= 8, "a register of first chunks");
    auto lane_offsets = [&](int64_t tile) __attribute__((always_inline)) {
        first_chunk = 0;
#pragma unroll
        for (int e = 0; e < LPW; ++e) {
            const int blk = wave * LPW + e;
            int ch = my_chunk(e);
            if (blk < C::A_BLK) {
                int64_t row = tile * BM + blk * RPB + lane / CPR;
                row = row < N ? row : N - 1;
                if constexpr (BY_LINE) {
                    asm volatile("" : "+v"(ch));          // (no register is left for what a ragged tile would find ready made)
                    ch = ((ch + lead(row)) & 7) - lead(row);
                }
                loff[e] = (uint32_t)(row - tile * BM) * (uint32_t)rb + ch * 16;
            } else {
                int q = n0 + (blk - C::A_BLK) * RPB + lane / CPR;
                q = q < B ? q : B - 1;
                loff[e] = (uint32_t)(q - n0) * (uint32_t)rb + ch * 16;
            }
            if constexpr (BY_LINE) first_chunk |= (uint32_t)(ch + 7) << (4 * e);
        }
    };
    auto offset = [&](int e) -> int64_t { return BY_LINE ? (int64_t)(int32_t)loff[e] : (int64_t)loff[e]; };
    auto chunk_of = [&](int e) { return BY_LINE ? (int)(first_chunk >> (4 * e) & 15) - 7 : my_chunk(e); };
    lane_offsets(t0);
    const char *xbase = static_cast<const char *>(X) + (size_t)t0 * BM * rb;              // tile start
    const char *qbase = static_cast<const char *>(Q) + (size_t)n0 * rb;
    const bool ragged_row = (rb & (SB - 1)) != 0;
    int iks = 0, issued = 0, iofs = 0;                   // k step and LDS offset of the next stage to issue
    int64_t itile = t0;
    constexpr bool LINES = SB == 128;
    const char *xs = xbase, *qs = qbase;                 // LINES: the next stage's place in them
    // LINES: inside a tile, before its last step
    auto issue_inside = [&]() __attribute__((always_inline)) {
        unsigned char *sbase = stage_mem + iofs;
#pragma unroll
        for (int e = 0; e < LPW; ++e) {
            const int blk = wave * LPW + e;
            ANN_GLOBAL_TO_LDS_16((blk < C::A_BLK ? xs : qs) + offset(e), sbase + blk * 1024);
        }
        iofs = iofs + C::STAGE_BYTES == C::LDS_BYTES ? 0 : iofs + C::STAGE_BYTES;
        xs += SB;
        qs += SB;
        ++issued;
        ++iks;
    };
    auto issue = [&]() __attribute__((always_inline)) {
        if (issued >= total) return;
        if (BY_LINE ? iks > 0 && 8 * iks + 7 < nch : LINES && iks < ksteps - 1) return issue_inside();
        ++issued;
        unsigned char *sbase = stage_mem + iofs;
        if (BY_LINE || (ragged_row && iks == ksteps - 1)) {
#pragma unroll
            for (int e = 0; e < LPW; ++e) {
                const int blk = wave * LPW + e;
                const char *base = blk < C::A_BLK ? xbase : qbase;
                const char *p = base + iks * SB + offset(e);
                const bool inside = (uint32_t)(iks * CPR + chunk_of(e)) < (uint32_t)nch;
                ANN_GLOBAL_TO_LDS_16(inside ? p : reinterpret_cast<const char *>(zero_row_end), sbase + blk * 1024);
            }
            if constexpr (BY_LINE) { xs += SB; qs += SB; }
        } else {
#pragma unroll
            for (int e = 0; e < LPW; ++e) {
                const int blk = wave * LPW + e;
                const char *base = blk < C::A_BLK ? xbase : qbase;
                ANN_GLOBAL_TO_LDS_16(base + iks * SB + offset(e), sbase + blk * 1024);
            }
        }
        iofs = iofs + C::STAGE_BYTES == C::LDS_BYTES ? 0 : iofs + C::STAGE_BYTES;
        if (++iks == lines) {
            iks = 0;
            ++itile;
            xbase += (size_t)BM * rb;
            if (LINES) { xs = xbase; qs = qbase; }
            if ((itile + 1) * BM > N && itile < t1) lane_offsets(itile);                  // ragged last tile
        }
    };

    f16v acc[WMF][WNF];
    int it = 0, cofs = 0;                                 // stage being computed, its LDS offset
    using Operands = u4[NKH][WMF + WNF];
    // the stage's operands; `inside` (LINES): there is a stage to load, and it lies inside its tile
    auto read = [&](Operands &x, auto inside) __attribute__((always_inline)) {
        // it has landed once only the newer stages' loads are outstanding (a tile's stores are newer still: the
        // wait right behind an epilogue is a little longer than it has to be)
        const int newer = decltype(inside)::value ? NST - 2 : min(NST - 2, total - 1 - it);
        if (newer == NST - 2) wait_vmcnt<(NST - 2) * LPW>();
        else static_for<NST - 2>([&](auto rc) {
            if (newer == decltype(rc)::value) wait_vmcnt<decltype(rc)::value * LPW>();
        });
        // ... for every wave.  And the buffer of stage it - 1 is free, which the next loads go to: no wave reads it any more.  Its products
        // see to that, which need what was read; BY_LINE they come a read later, so the reads are waited for (a tile's first line: its
        // second one is read before any product).
        if constexpr (BY_LINE) barrier_after_reads();
        else bare_barrier();
        if constexpr (!LINES) issue();
        // Operand row r = lane % 32 of a 32-row block pair, chunk 2 kh + lane / 32.  All operand reads of the stage
        // are issued before the first MFMA, so the LDS pipeline always has several 1 KB reads of this wave in flight.
        const unsigned char *sb = stage_mem + cofs;
#pragma unroll
        for (int kh = 0; kh < NKH; ++kh) {
            const int lofs = (l32 / RPB) * 1024 + (l32 & (RPB - 1)) * SB + (((2 * kh + lhi) ^ swz(l32)) * 16);
#pragma unroll
            for (int j = 0; j < WNF; ++j)
                x[kh][WMF + j] = *reinterpret_cast<const u4 *>(sb + (C::A_BLK + (wn * WNF + j) * (32 / RPB)) * 1024 + lofs);
#pragma unroll
            for (int i = 0; i < WMF; ++i)
                x[kh][i] = *reinterpret_cast<const u4 *>(sb + (wm * WMF + i) * (32 / RPB) * 1024 + lofs);
        }
        if constexpr (LINES) {                            // (the addresses are made while the reads run)
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (decltype(inside)::value) issue_inside();
            else issue();
        }
        __builtin_amdgcn_sched_barrier(0);                // keep the reads ahead of the MFMAs
        cofs = cofs + C::STAGE_BYTES == C::LDS_BYTES ? 0 : cofs + C::STAGE_BYTES;
        ++it;
    };
    auto multiply = [&](Operands &x, auto first) __attribute__((always_inline)) {
        static_for<NKH>([&](auto kc) {
            static_for<WMF>([&](auto ic) {
                static_for<WNF>([&](auto jc) {
                    constexpr int kh = decltype(kc)::value, i = decltype(ic)::value, j = decltype(jc)::value;
                    if constexpr (decltype(first)::value && kh == 0) {
                        f16v zero;
#pragma unroll
                        for (int r = 0; r < 16; ++r) zero[r] = 0.f;
                        acc[i][j] = mfma32<T>(x[kh][i], x[kh][WMF + j], zero);
                    } else {
                        acc[i][j] = mfma32<T>(x[kh][i], x[kh][WMF + j], acc[i][j]);
                    }
                });
            });
        });
    };
    auto stage = [&](auto first, auto inside) __attribute__((always_inline)) {
        Operands x;
        read(x, inside);
        multiply(x, first);
    };
    // BY_LINE: the LDS place of chunk 2 kh + lane / 32 of a step holds, of the line as many stages into the tile, that chunk if kh < keep,
    // else that of the step before.  So the products of a step follow the reads of the next line.
    int keep[WMF];
    if constexpr (BY_LINE) {
#pragma unroll
        for (int i = 0; i < WMF; ++i) keep[i] = 4 - ((lead((wm * WMF + i) * 32 + l32) + lhi) >> 1);
    }
    // the corpus operands of a step, in `x` as its own line had them: the rest from `next`, the line after it, or zeros behind the last one
    auto complete = [&](Operands &x, const Operands &next, auto end) __attribute__((always_inline)) {
#pragma unroll
        for (int kh = 0; kh < NKH; ++kh)
#pragma unroll
            for (int i = 0; i < WMF; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c) x[kh][i][c] = kh < keep[i] ? x[kh][i][c] : decltype(end)::value ? 0u : next[kh][i][c];
    };
    // the next line into `y`, and the products of the step that `x` was read for
    auto line = [&](Operands &x, Operands &y, auto first, auto inside) __attribute__((always_inline)) {
        read(y, inside);
        complete(x, y, std::false_type{});
        multiply(x, first);
    };

    for (int s = 0; s < NST - 1; ++s) issue();
    for (int64_t tile = t0; tile < t1; ++tile) {
        if constexpr (BY_LINE) {                          // (rows of more than a line: at least two stages)
            Operands u, v;
            read(u, std::false_type{});
            line(u, v, std::true_type{}, std::false_type{});
            int j = 2;
            // pairs of lines that need no look at where the loads are, which are not in a tile's first line
            for (int n = iks > 0 ? min((nch >> 3) - iks, total - issued) >> 1 : 0; n > 0; --n, j += 2) {
                line(v, u, std::false_type{}, std::true_type{});
                line(u, v, std::false_type{}, std::true_type{});
            }
            for (; j + 1 < lines; j += 2) {
                line(v, u, std::false_type{}, std::false_type{});
                line(u, v, std::false_type{}, std::false_type{});
            }
            auto flush = [&](Operands &x) __attribute__((always_inline)) {
                if (lines != ksteps) return;              // (else the last line ends the last step)
                complete(x, x, std::true_type{});
                multiply(x, std::false_type{});
            };
            if (j < lines) {
                line(v, u, std::false_type{}, std::false_type{});
                flush(u);
            } else {
                flush(v);
            }
        } else {
            stage(std::true_type{}, std::false_type{});
            for (int ks = 1; ks < ksteps;) {
                if constexpr (LINES) {                    // steps that need no look at where the loads are
                    int n = min(min(ksteps - ks, ksteps - 1 - iks), total - issued);
                    ks += max(n, 0);
                    for (; n > 0; --n) stage(std::false_type{}, std::true_type{});
                    if (ks == ksteps) break;
                }
                stage(std::false_type{}, std::false_type{});
                ++ks;
            }
        }

        int ln = lane;
        asm volatile("" : "+v"(ln));                      // (nothing of the epilogue is worth a register in the loop above)
        const int l32 = ln & 31, lhi = ln >> 5;
        const int rbase = (int)(tile * BM) + wm * 32 * WMF + 4 * lhi;     // N < 2^31
        const int nrows = (int)N;
        if ((tile + 1) * BM > N) {
            static_for<WMF>([&](auto ic) {
                static_for<WNF>([&](auto jc) {
                    constexpr int i = decltype(ic)::value, j = decltype(jc)::value;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (rbase + (i * 32 + 8 * (r / 4) + (r % 4)) >= nrows) acc[i][j][r] = __builtin_nanf("");
                });
            });
        }
        // Where the part starts is added only where a boundary is: left to itself the compiler takes the sum out of the
        // branch and keeps a second set of row numbers for every search, 0.15 us of the 12.6 of 1024 rows x 768, B = 512.
        auto part_start = [&] { int b = after.base; asm volatile("" : "+s"(b)); return b; };
        static_for<WNF>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const int q = n0 + (wn * WNF + j) * 32 + l32;
            if (after.s) {                                // rows at or before the query's boundary do not take part
                const float bs = after.s[min(q, B - 1)];
                const int bid = after.id[min(q, B - 1)], rafter = rbase + part_start();
                static_for<WMF>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        acc[i][j][r] = after_boundary(acc[i][j][r], rafter + (i * 32 + 8 * (r / 4) + (r % 4)), bs, bid);
                });
            }
            if constexpr (ONE) {
                if (tile + 1 == t1 && B > 64) {
                    // The stages are free: through LDS, so that a store writes whole lines, past the L2 (from the registers
                    // it is 16 bytes to each of 64 lines, and 20 MB of them wait for the end of the kernel: 977 x 64, B = 5000
                    // 16.9 -> 11.9 us; 3224 x 576, B = 3326 51 -> 41.5).  Few queries do without the barrier (4364 x 608, B = 28
                    // 12.6, 12.9 through LDS).
                    if constexpr (j == 0) bare_barrier();     // every wave has read the last stage
                    constexpr int U = WMF < 2 ? WMF : 2, ROW = 32 * U + 4, UNITS = 8 * U;
                    static_assert(32 * ROW * 4 <= C::LDS_BYTES / C::WAVES, "a wave's share of the stages");
                    float *own = reinterpret_cast<float *>(stage_mem) + wave * (C::LDS_BYTES / C::WAVES / 4);
                    static_for<WMF / U>([&](auto pc) {
                        constexpr int i0 = decltype(pc)::value * U;
                        static_for<U>([&](auto uc) {
                            constexpr int i = i0 + decltype(uc)::value, u = decltype(uc)::value;
#pragma unroll
                            for (int r = 0; r < 16; r += 4)
                                *reinterpret_cast<f4 *>(own + l32 * ROW + lhi * 16 * U + u * 16 + r) =
                                    f4{acc[i][j][r], acc[i][j][r + 1], acc[i][j][r + 2], acc[i][j][r + 3]};
                        });
                        float *o = maxima + tile * BM + i0 * 16;
#pragma unroll
                        for (int e = 0; e < 32 * UNITS / 64; ++e) {
                            const int row = (e * 64 + ln) / UNITS, unit = ln % UNITS;
                            const int qr = n0 + (wn * WNF + j) * 32 + row;
                            const f4 v = *reinterpret_cast<const f4 *>(own + row * ROW + unit * 4);
                            const int at = (wm * 2 + unit / (4 * U)) * (16 * WMF) + unit % (4 * U) * 4;
                            if (qr < B) __builtin_nontemporal_store(v, reinterpret_cast<f4 *>(o + (size_t)qr * n + at));
                        }
                    });
                } else if (q < B) {
                    float *o = maxima + (size_t)q * n + (size_t)tile * BM + (wm * 2 + lhi) * (16 * WMF);
                    static_for<WMF>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
#pragma unroll
                        for (int r = 0; r < 16; r += 4)
                            *reinterpret_cast<f4 *>(o + i * 16 + r) =
                                f4{acc[i][j][r], acc[i][j][r + 1], acc[i][j][r + 2], acc[i][j][r + 3]};
                    });
                }
            } else if (q < B) {
                // this lane's groups of the tile, side by side
                float *o = maxima + (size_t)q * n + (((size_t)tile * BM + (wm * 2 + lhi) * (16 * WMF)) >> gs_log);
                float m16[WMF];
                static_for<WMF>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    f4 m;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        m[u] = fmaxf(fmaxf(acc[i][j][4 * u], acc[i][j][4 * u + 1]),
                                     fmaxf(acc[i][j][4 * u + 2], acc[i][j][4 * u + 3]));
                    if (gs_log == 2) *reinterpret_cast<f4 *>(o + i * 4) = m;
                    m16[i] = fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
                });
                if (gs_log == 4) {
#pragma unroll
                    for (int i = 0; i < WMF; ++i) o[i] = m16[i];
                } else if (gs_log == 5) {
                    if constexpr (WMF >= 2) static_for<WMF / 2>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        o[i] = fmaxf(m16[2 * i], m16[2 * i + 1]);
                    });
                } else if (gs_log == 6) {
                    if constexpr (WMF == 4) *o = fmaxf(fmaxf(m16[0], m16[1]), fmaxf(m16[2], m16[3]));
                }
            }
        });
    }
}

}  // namespace ann

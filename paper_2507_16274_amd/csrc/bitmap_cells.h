// What the two occupancy-bitmap kernels share: the table cell of a placed block, marking blocks in a bitmap in
// LDS, and the search for a run of free granules.
#pragma once

#include <type_traits>

#include "host_util.h"
#include "wave.h"

namespace stalloc {

constexpr int kRowPad = 256;             // index rows are padded to this many entries (4 per lane)
constexpr uint32_t kBmMaxRequests = 32768;         // index entries are 16-bit request numbers; the index has n^2 of them at worst

// Entries are 4 * j, the byte offset into the plan's table, while that fits 16 bits, else j.
constexpr uint32_t kScaledEntriesBelow = 16384;
__host__ __device__ inline uint32_t entry_shift(uint32_t n) { return n < kScaledEntriesBelow ? 2u : 0u; }

// A placed block as the build phase wants it: bits 0-21 address in granules (bits 0-4 = first bit
// b in its first word, bits 5-21 = that word), bits 22-26 size in granules (1..31), bits 27-31 the
// number of granules that spill into the next word.  0 = not placed.
constexpr uint32_t kCellSizeAt = 22, kCellSpillAt = 27;
__device__ __forceinline__ uint32_t make_cell(uint32_t x, uint32_t sz)
{
    const uint32_t reach = (x & 31) + sz;
    return x | (sz << kCellSizeAt) | ((reach > 32 ? reach - 32 : 0u) << kCellSpillAt);
}

// ((1 << width) - 1) << offset with both taken modulo 32.
__device__ __forceinline__ uint32_t bit_field_mask(uint32_t width, uint32_t offset)
{
    uint32_t r;
    asm("v_bfm_b32 %0, %1, %2" : "=v"(r) : "v"(width), "v"(offset));
    return r;
}

typedef __attribute__((address_space(3))) uint32_t lds_word;

// LDS address of the first bitmap word of the block of `cell`: field extract, shift-add.
__device__ __forceinline__ lds_word* first_word(uint32_t* bm, uint32_t cell)
{
    const uint32_t base = (uint32_t)reinterpret_cast<uintptr_t>((lds_word*)bm);
    uint32_t at;
    asm("v_bfe_u32 %0, %1, 5, 17\n\tv_lshl_add_u32 %0, %0, 2, %2" : "=&v"(at) : "v"(cell), "s"(base));
    return reinterpret_cast<lds_word*>((uintptr_t)at);
}

// ORs the block of `cell` into the bitmap; cell == 0 adds nothing.
__device__ __forceinline__ void mark_cell(uint32_t* bm, uint32_t cell)
{
    lds_word* word = first_word(bm, cell);
    const uint32_t first = bit_field_mask(cell >> kCellSizeAt, cell);      // ((1 << size) - 1) << b, low 32 bits
    const uint32_t spill = bit_field_mask(cell >> kCellSpillAt, 0u);       // (1 << spilled) - 1
    if (cell) __hip_atomic_fetch_or(word, first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (cell >= (1u << kCellSpillAt)) __hip_atomic_fetch_or(word + 1, spill, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The same for four cells per lane, looking before ORing.  Blocks that are alive at different
// times share addresses (that is the point of the plan), so most blocks of a row only repeat
// bits that are already set, and many lanes of one instruction aim at the same few words.  LDS
// serialises atomics on one address lane by lane but broadcasts reads of one address, hence:
// read the words, and send only the lanes that still add a bit into the atomic.  (A word read
// just before another wave's OR merely causes a redundant OR.)  Address and masks are worked
// out for every lane; idle lanes have empty masks and drop out with the rest.
__device__ __forceinline__ void mark_cells(uint32_t* bm, const uint32_t (&cell)[4])
{
    lds_word* word[4];
    uint32_t first[4], spill[4], seen[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        word[k] = first_word(bm, cell[k]);
        first[k] = bit_field_mask(cell[k] >> kCellSizeAt, cell[k]);
        spill[k] = bit_field_mask(cell[k] >> kCellSpillAt, 0u);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) seen[k] = *word[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (first[k] & ~seen[k]) __hip_atomic_fetch_or(word[k], first[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cell[k] >= (1u << kCellSpillAt)) __hip_atomic_fetch_or(word[k] + 1, spill[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// Lowest bit position x >= 32 * first such that bits [x, x + s) of the bitmap are zero; words at and beyond
// `limit` count as free.  1 <= s <= 32, s, first and limit uniform.  Whole wave, uniform result.
__device__ __forceinline__ uint32_t first_fit(const uint32_t* bm, uint32_t limit, uint32_t s, uint32_t first = 0)
{
    const int lane = lane_id();
    for (uint32_t t = first;; t += kWave) {
        const uint32_t w = t + lane;
        const uint32_t here = w < limit ? bm[w] : 0u;
        const uint32_t next = w + 1 < limit ? bm[w + 1] : 0u;
        uint64_t free_run = ~((uint64_t)here | ((uint64_t)next << 32));     // bit b: granule 32 w + b is free
        for (uint32_t len = 1; len < s;) {                                  // bit b: free for `len` granules from b
            const uint32_t step = len < s - len ? len : s - len;
            free_run &= free_run >> step;
            len += step;
        }
        const uint32_t starts = (uint32_t)free_run;                         // runs that begin inside word w
        const uint64_t any = __builtin_amdgcn_uicmp(starts, 0u, 33);        // != 0
        if (any) {
            const int f = __builtin_ctzll(any);
            return (t + (uint32_t)f) * 32 + (uint32_t)__builtin_ctz(read_lane(starts, f));
        }
    }
}

// Lowest fit of a request of s granules among the 64 granules from the word of its candidate x on (`word`: how its bitmap has
// them), if the blocks of the lanes in `rivals` are there as well, each ((1 << size) - 1 = ones) from granule lo on; kNoFit if there is
// none.  The blocks become bits in their lanes, those are ORed over the wave, and the search goes on in scalar registers: nothing
// here waits for LDS, and a lone wave, which issues an instruction every six cycles or so, gets by with some seventy.
constexpr uint32_t kNoFit = 0xffffffffu;
__device__ __forceinline__ uint32_t fit_among(uint64_t word, uint32_t s, uint32_t x, uint64_t rivals, uint32_t lo, uint32_t ones)
{
    const uint32_t base = x & ~31u;
    // the 64 bits from the word before on hold what reaches into the first word, the 64 from the first on what reaches into the second
    const uint32_t up = lo + (32u - base), on = lo - base;
    const uint32_t in_first = lane_in(rivals & lanes_lt(up, 64u)) ? ones : 0u, in_second = lane_in(rivals & lanes_lt(on, 64u)) ? ones : 0u;
    uint32_t u = (uint32_t)(((uint64_t)in_first << (up & 63u)) >> 32), v = (uint32_t)(((uint64_t)in_second << (on & 63u)) >> 32);
    auto both = [&](auto ctrl, auto rows) {
        u |= __builtin_amdgcn_update_dpp(0u, u, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        v |= __builtin_amdgcn_update_dpp(0u, v, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
    };
    both(std::integral_constant<int, kDppRowShr1>(), std::integral_constant<int, 0xf>());
    both(std::integral_constant<int, kDppRowShr2>(), std::integral_constant<int, 0xf>());
    both(std::integral_constant<int, kDppRowShr4>(), std::integral_constant<int, 0xf>());
    both(std::integral_constant<int, kDppRowShr8>(), std::integral_constant<int, 0xf>());
    both(std::integral_constant<int, kDppRowBcast15>(), std::integral_constant<int, 0xa>());
    both(std::integral_constant<int, kDppRowBcast31>(), std::integral_constant<int, 0xc>());
    const uint64_t rest = ((uint64_t)read_lane(v, kWave - 1) << 32) | read_lane(u, kWave - 1);
    uint64_t free_run = ~(word | rest);
    for (uint32_t len = 1; len < s;) {                                       // bit b: free for `len` granules from b, all of them in the 64
        const uint32_t step = len < s - len ? len : s - len;
        free_run &= free_run >> step;
        len += step;
    }
    return free_run ? base + (uint32_t)__builtin_ctzll(free_run) : kNoFit;
}

// Fills the row of one request with the requests j for which listed(j) holds; called by a workgroup of 256
// threads with `room` entries to write to; returns how many there are, entries that do not fit included.
// The order of a row's entries is free (the bitmap is an OR over the row), so it is chosen for the
// table lookups of the build phase: one lookup instruction reads the table cells of 64 consecutive
// entries of this order, and LDS serves them fastest when they lie in different banks (cell j is
// in bank j mod 32).  Entries are ordered by (rank, bank), rank = how many entries of the same bank
// come before: any 64 in a row then hold every bank about twice.  Within a chunk of 256, entry e
// belongs to lane e / 4 and lookup e mod 4, hence the transposition.  Places up to the next multiple
// of 256 (at most `room`) are filled with n, a request that is never placed.
struct RowLds {
    static constexpr uint32_t kMaxRank = kBmMaxRequests / 32;
    uint32_t per_thread[256];
    uint32_t in_bank[32];
    uint32_t before_rank[kMaxRank + 1];      // entries with a lower rank
    uint32_t banks_at_rank[kMaxRank + 1];    // banks that have an entry of this rank
};
template <typename Listed>
__device__ __forceinline__ uint32_t fill_row(uint16_t* row, uint32_t room, uint32_t n, RowLds& sh, Listed&& listed)
{
    const uint32_t t = threadIdx.x;
    const uint32_t bank = t & 31u;                      // thread t sees j = t, t + 256, ...: all in one bank
    uint32_t mine = 0;
    for (uint32_t j = t; j < n; j += 256) mine += listed(j) ? 1u : 0u;
    sh.per_thread[t] = mine;
    __syncthreads();
    uint32_t rank = 0, total = 0;                       // of the 8 threads of a bank, the lower ones come first
    for (uint32_t m = 0; m < 8; ++m) {
        const uint32_t c = sh.per_thread[bank + 32 * m];
        if (m < (t >> 5)) rank += c;
        total += c;
    }
    if (t < 32) sh.in_bank[t] = total;
    __syncthreads();
    for (uint32_t r = t; r <= RowLds::kMaxRank; r += 256) {
        uint32_t before = 0, banks = 0;
        for (uint32_t b = 0; b < 32; ++b) {
            const uint32_t c = sh.in_bank[b];
            before += c < r ? c : r;
            banks |= (c > r ? 1u : 0u) << b;
        }
        sh.before_rank[r] = before;
        sh.banks_at_rank[r] = banks;
    }
    __syncthreads();
    auto slot = [](uint32_t pos) {                      // position in the order -> entry of the row
        const uint32_t p = pos % kRowPad;
        return pos - p + 4 * (p % kWave) + p / kWave;
    };
    for (uint32_t j = t; j < n; j += 256) {
        if (listed(j)) {
            const uint32_t pos = sh.before_rank[rank] + (uint32_t)__builtin_popcount(sh.banks_at_rank[rank] & ((1u << bank) - 1u));
            if (pos < room) row[slot(pos)] = (uint16_t)(j << entry_shift(n));
            ++rank;
        }
    }
    const uint32_t filled = sh.before_rank[RowLds::kMaxRank];      // = number of entries
    uint32_t end = (filled + kRowPad - 1) / kRowPad * kRowPad;
    if (end > room) end = room;
    for (uint32_t pos = filled + t; pos < end; pos += 256) row[slot(pos)] = (uint16_t)(n << entry_shift(n));
    return filled;
}

}  // namespace stalloc

// kernels.hip -- gfx950 kernels of libckpt: size scan, chunk map, fused
// pack + CRC-32C + ZERO/DIRTY flags (and its hash-only and restore/verify
// variants), selection scan, gather, and small helpers.
//
// The data path drains the memory of live allocations into an image and
// refills it (CRAC, Sec. 3.2 "Saving the library-allocated arena" and
// "restoring the CUDA library-allocated regions").  It is pure bandwidth
// work: no MFMA.  The CRC-32C per chunk is the library's own check.
//
// CRC scheme (one wave64 per chunk, or `waves_per_chunk` waves):
//   * The chunk's bytes are read in rounds of 1 KiB: in round r, lane l loads
//     the 16-byte piece r*64 + l (each load instruction covers 1 KiB of whole
//     cache lines).
//   * A chunk of len bytes is placed at the END of a window of whole rounds
//     (leading zero pieces, and zeros after len up to the next 16 bytes).
//     Leading zeros leave a zero CRC register unchanged, so the window's raw
//     CRC (zero init, no final XOR) equals that of the data followed by its
//     s = roundup16(len) - len zero pad bytes; the pad is undone at the end by
//     the inverse operator for s bytes.
//   * Each lane hashes each round's piece from a zero register (two 2-byte
//     table steps per 4-byte word) and combines the rounds by Horner's rule
//     with the one-round operator (1024 - 16 bytes to the lane's next piece).
//   * A 6-level tree across lanes combines the registers: at level k the left
//     partner is moved forward 16 << k bytes and XORed with the right one;
//     only the lanes whose result is still needed do the table lookups.
//   * With several waves per chunk, each wave owns consecutive rounds and the
//     per-wave results are combined by one more operator.
//   * CRC-32C's initial value 0xFFFFFFFF is folded in by complementing the
//     first min(len, 4) data bytes before hashing (and, for len < 4, XORing
//     the part of the initial value that is still in the register), and the
//     final XOR is applied last.
//   Every "move forward m bytes" is a GF(2)-linear operator stored in LDS as
//   byte-indexed tables (crc_tables.cpp), the chain and round operators
//   replicated per lane so that the random lookups are bank-conflict free.
#include "internal.h"

namespace ckpt {

// ------------------------------------------------------------------ helpers

__device__ __forceinline__ uint32_t apply_op(const uint32_t *__restrict__ t, uint32_t v)
{
    return t[v & 0xffu] ^ t[256 + ((v >> 8) & 0xffu)] ^ t[512 + ((v >> 16) & 0xffu)] ^
           t[768 + (v >> 24)];
}

// The operator tables as staged in LDS (126 KiB): per-lane copies of the
// chain and round operators, single copies of the tree and cross-wave ones.
struct Tabs {
    const uint32_t *t;   // LDS base
    uint32_t lb;         // (lane & 31) << 2, this lane's chain copy
    uint32_t lb8;        // (lane & 7) << 2, this lane's round-operator copy

    __device__ __forceinline__ uint32_t lds(uint32_t byte_off) const
    {
        return *(const uint32_t *)((const uint8_t *)t + byte_off);
    }
    // the two lookups of a 2-byte step of register y, which then is *t0 ^ *t1 ^ (y >> 16)
    __device__ __forceinline__ void chain_lookups(uint32_t y, uint32_t *t0, uint32_t *t1) const
    {
        const uint32_t a0 = __builtin_amdgcn_perm(y, lb, 0x0c0c0400u);   // (y.byte0 << 8) | lb
        const uint32_t a1 = (y & 0xff00u) | lb;
        *t0 = lds(kRepChainOff + a0);
        *t1 = lds(kRepChainOff + 128 + a1);
    }
    // register after the 4-byte word w: two 2-byte steps
    __device__ __forceinline__ uint32_t chain(uint32_t s, uint32_t w) const
    {
        uint32_t y = s ^ w;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            uint32_t t0, t1;
            chain_lookups(y, &t0, &t1);
            y = t0 ^ t1 ^ (y >> 16);
        }
        return y;
    }
    // the register moved one round (or, in the quad form's set, the skip) forward
    __device__ __forceinline__ uint32_t gap(uint32_t v) const
    {
        return lds(((v & 0xffu) << 5) | lb8) ^ lds(8192 + ((((v >> 8) & 0xffu) << 5) | lb8)) ^
               lds(16384 + ((((v >> 16) & 0xffu) << 5) | lb8)) ^ lds(24576 + (((v >> 24) << 5) | lb8));
    }
    __device__ __forceinline__ uint32_t tree(int k, uint32_t v) const
    {
        return apply_op(t + kRepTreeOff / 4 + k * kTabWords, v);
    }
    __device__ __forceinline__ uint32_t seg(uint32_t v) const
    {
        return apply_op(t + kRepTreeOff / 4 + kTreeLevels * kTabWords, v);
    }
};

__device__ __forceinline__ Tabs make_tabs(const uint32_t *lds_tabs, int lane)
{
    Tabs T;
    T.t = lds_tabs;
    T.lb = (uint32_t)(lane & 31) << 2;
    T.lb8 = (uint32_t)(lane & 7) << 2;
    return T;
}

// The first lane's value, for the whole wave.
__device__ __forceinline__ uint32_t uniform_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v)
{
    return ((uint64_t)uniform_u32((uint32_t)(v >> 32)) << 32) | uniform_u32((uint32_t)v);
}

__device__ __forceinline__ uint64_t round_up16(uint64_t x) { return (x + 15) & ~uint64_t(15); }

// Wave64 inclusive scan of a u64 (Hillis-Steele with shuffles).
__device__ __forceinline__ uint64_t wave_incl_scan(uint64_t v, int lane)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint64_t o = __shfl_up(v, d, 64);
        if (lane >= d) v += o;
    }
    return v;
}

// v with its bytes from `valid` on (0 < valid < 16) cleared.
__device__ __forceinline__ uint4 keep_bytes(uint4 v, uint32_t valid)
{
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (uint32_t i = 0; i < 4; i++)
        w[i] &= valid >= 4 * i + 4 ? 0xFFFFFFFFu : valid <= 4 * i ? 0u : (1u << (8 * (valid - 4 * i))) - 1u;
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// The chunks' addresses are integers in their descriptors, and a pointer made
// from one is generic: the compiler accesses it with flat instructions, which
// count as LDS accesses too, so every wait for a table lookup also waited for
// the next chunk's loads and for the stores before it.  These say that the
// address is of device or host memory, never LDS.  (8 GiB snapshot 2.28 ->
// 2.20 ms, 4 GiB of random 4 KiB chunks 1.51 -> 1.44 - 1.48 ms, both with
// arrived() below; 16384 allocations of 16 B to 32 KiB, pack kernel 51 ->
// 42 us with the one-wave form's cuts moved behind the loads.)
template <class T>
using Global = __attribute__((address_space(1))) T;
template <class T>
using Local = __attribute__((address_space(3))) T;

// Writes bytes [0, valid) of a 16-byte piece only (q 16-byte aligned).
__device__ __forceinline__ void store_partial(uint8_t *q, uint32_t valid, uint4 v)
{
    Global<uint8_t> *p = (Global<uint8_t> *)q;
    uint32_t lo = v.x, hi = v.y;   // the 8 bytes not yet written
    if (valid & 8) {
        *(Global<uint64_t> *)p = (uint64_t)hi << 32 | lo;
        lo = v.z;
        hi = v.w;
    }
    if (valid & 4) {
        *(Global<uint32_t> *)(p + (valid & 8)) = lo;
        lo = hi;
    }
    if (valid & 2) {
        *(Global<uint16_t> *)(p + (valid & 12)) = (uint16_t)lo;
        lo >>= 16;
    }
    if (valid & 1)
        p[valid & 14] = (uint8_t)lo;
}

// XOR of the 16 lanes of a row, in each of them (DPP: lanes 1, then 2 apart,
// then the mirrored half row and row).
__device__ __forceinline__ uint32_t row_xor(uint32_t x)
{
    x ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true);
    x ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true);
    x ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true);
    x ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, true);
    return x;
}

// Undo `s` zero pad bytes (0 < s < 16) of a register that all lanes of a row
// hold: the inverse operator's columns at the register's set bits, two
// columns per lane.  (Bit by bit in one lane these are up to 120 dependent
// steps, and a tail read byte by byte 15 loads: with both, a snapshot of 16384
// allocations of odd sizes up to 32 KiB took 241 us, now 206.)
__device__ __forceinline__ uint32_t row_unshift(const Tabs &T, uint32_t reg, uint32_t s, int lane)
{
    const uint32_t lr = (uint32_t)lane & 15;
    const uint32_t at = kRepUnshiftOff + ((s - 1) * 32 + lr) * 4;
    const uint32_t c0 = T.lds(at), c1 = T.lds(at + 64);
    return row_xor(((reg >> lr) & 1u ? c0 : 0u) ^ ((reg >> (lr + 16)) & 1u ? c1 : 0u));
}

// Mask that complements the first min(n, 4) bytes of the first data word.
__device__ __forceinline__ uint32_t init_mask(uint32_t n)
{
    return n >= 4 ? 0xFFFFFFFFu : ((1u << (8 * n)) - 1u);
}

// CRC-32C from the window's raw register, which (like n) every lane of a row
// holds; the rows of a wave may hold different chunks.  The whole wave must be
// active.
__device__ __forceinline__ uint32_t finish_crc(const Tabs &T, uint32_t raw, uint32_t n, int lane)
{
    const uint32_t s = (0u - n) & 15u;
    uint32_t reg = raw;
    if (__ballot(s != 0)) {   // else every chunk of the wave ends on a piece
        const uint32_t r = row_unshift(T, raw, s ? s : 1u, lane);
        reg = s ? r : raw;
    }
    if (n < 4)
        reg ^= 0xFFFFFFFFu >> (8 * n);
    return ~reg;
}

// ---------------------------------------- K1: size scan and chunk -> row map
//
// off[k] = exclusive prefix sum of roundup16(size), cb[k] = exclusive prefix
// sum of ceil(size / C), off[n] and cb[n] the totals; map[g] = k for every
// chunk g of allocation k: the descriptor table each workgroup of the chunk
// kernels stages into LDS, one load per chunk instead of a binary search.
//
// The host lays the table out in pinned memory (TableUpload): a plan header,
// the addresses and sizes, for every kRowTile rows the offsets their scan
// starts from, and the pieces that allocations of more than kBigRow chunks
// are cut into for the map.  One launch reads it across the host link and
// does everything: a work item is a tile of rows (read, scanned by one wave,
// its short rows mapped by the workgroup) or a piece of a long row.  Bound by
// latency.  One workgroup that walked the table in tiles of 1024, then a map
// launch with a wave per row, took 71 us for 16384 rows, 26 us for 4096, and
// for one allocation of 10^6 chunks the map alone about 300 us.

constexpr int kPrologueThreads = 256;

__device__ __forceinline__ void map_range(uint32_t *__restrict__ map, uint64_t g, uint64_t end, uint64_t step,
                                          uint32_t k)
{
    for (; g < end; g += step)
        map[g] = k;
}

// Rows [first, first + kRowTile) by the first wave: size and address at hand,
// the prefix sums starting from (o, c).  s_cb gets the rows' first chunks.
__device__ __forceinline__ void scan_rows(const PrologueArgs &a, uint64_t n, uint64_t first, int lane, uint64_t ad,
                                          uint64_t sz, uint64_t o, uint64_t c, uint64_t *s_cb)
{
    const uint64_t k = first + lane;
    const uint64_t e = round_up16(sz), nc = (sz + a.C - 1) / a.C;
    const uint64_t ie = wave_incl_scan(e, lane), ic = wave_incl_scan(nc, lane);
    if (k < n) {
        a.addr[k] = ad;
        a.size[k] = sz;
        a.off[k] = o + ie - e;
        a.cb[k] = c + ic - nc;
        if (k + 1 == n) {
            a.off[n] = o + ie;
            a.cb[n] = c + ic;
        }
    }
    s_cb[lane] = c + ic - nc;
    if (lane == 63)
        s_cb[kRowTile] = c + ic;
}

// Thread `me` of `all` copies its share of a span.
__device__ __forceinline__ void copy_span(const CopySpan &x, uint64_t me, uint64_t all)
{
    const uint32_t odd = (uint32_t)((uintptr_t)x.src | (uintptr_t)x.dst);   // sections share a block
    uint64_t done = 0;
    if ((odd & 15) == 0) {
        for (uint64_t i = me; i < x.bytes / 16; i += all)
            ((uint4 *)x.dst)[i] = ((const uint4 *)x.src)[i];
        done = x.bytes / 16 * 16;
    } else if ((odd & 3) == 0) {
        for (uint64_t i = me; i < x.bytes / 4; i += all)
            ((uint32_t *)x.dst)[i] = ((const uint32_t *)x.src)[i];
        done = x.bytes / 4 * 4;
    }
    for (uint64_t i = done + me; i < x.bytes; i += all)
        ((uint8_t *)x.dst)[i] = ((const uint8_t *)x.src)[i];
}

__global__ __launch_bounds__(kPrologueThreads) void k_prologue(PrologueArgs a)
{
    __shared__ uint64_t s_cb[kRowTile + 1];
    const uint64_t n = a.n_known ? a.n_known : a.up_plan->n_allocs;
    const uint64_t np = a.n_known ? a.pieces_known : a.up_plan->n_pieces;
    const uint64_t tiles = (n + kRowTile - 1) / kRowTile;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = kPrologueThreads / 64;
    if (blockIdx.x == 0 && threadIdx.x < sizeof(DevPlan) / 8)
        ((uint64_t *)a.plan)[threadIdx.x] = ((const uint64_t *)a.up_plan)[threadIdx.x];
    for (uint64_t i = (uint64_t)blockIdx.x * kPrologueThreads + threadIdx.x; i < a.zero_words;
         i += (uint64_t)gridDim.x * kPrologueThreads)
        a.zero[i] = 0;
    for (uint32_t c = 0; c < a.n_copy; c++)
        copy_span(a.copy[c], (uint64_t)blockIdx.x * kPrologueThreads + threadIdx.x,
                  (uint64_t)gridDim.x * kPrologueThreads);
    for (uint64_t i = blockIdx.x; i < tiles + np; i += gridDim.x) {   // uniform over the workgroup
        if (i >= tiles) {
            const MapPiece pc = a.up_pieces[i - tiles];
            map_range(a.map, pc.begin + threadIdx.x, pc.end, kPrologueThreads, (uint32_t)pc.row);
            continue;
        }
        const uint64_t first = i * kRowTile;
        if (wave == 0) {
            const uint64_t k = first + lane;
            const uint64_t ad = k < n ? a.up_addr[k] : 0, sz = k < n ? a.up_size[k] : 0;
            scan_rows(a, n, first, lane, ad, sz, a.up_base[2 * i], a.up_base[2 * i + 1], s_cb);
        }
        __syncthreads();
        for (int r = wave; r < kRowTile; r += nw)
            if (s_cb[r + 1] - s_cb[r] <= kBigRow)
                map_range(a.map, s_cb[r] + lane, s_cb[r + 1], 64, (uint32_t)(first + r));
        __syncthreads();   // s_cb is rewritten
    }
}

// The same for a table of at most kRowTile rows that comes in the kernel's
// arguments (the allocation-free path): one workgroup, no host memory read.
__global__ __launch_bounds__(1024) void k_prologue_small(PrologueArgs a, SmallTable t)
{
    __shared__ uint64_t s_cb[kRowTile + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint64_t n = a.n_known;
    if (threadIdx.x == 64) {
        DevPlan p = {};
        p.n_allocs = n;
        p.n_chunks = t.n_chunks;
        p.data_bytes = t.data_bytes;
        *a.plan = p;
    }
    if (wave == 0)
        scan_rows(a, n, 0, lane, (uint64_t)lane < n ? t.addr[lane] : 0, (uint64_t)lane < n ? t.size[lane] : 0, 0, 0,
                  s_cb);
    __syncthreads();
    for (int r = 0; r < (int)n; r++)
        if (s_cb[r + 1] - s_cb[r] > kBigRow)
            map_range(a.map, s_cb[r] + threadIdx.x, s_cb[r + 1], blockDim.x, (uint32_t)r);
        else if (r % nw == wave)
            map_range(a.map, s_cb[r] + lane, s_cb[r + 1], 64, (uint32_t)r);
}

// The scan alone, over a table on the device (plan and size): one workgroup
// of 1024 threads walks it in tiles of 1024, then k_chunk_map.  For
// allocation-free calls with more rows than arguments hold.
__global__ __launch_bounds__(1024) void k_layout_scan(DevPlan *plan, const uint64_t *__restrict__ size, uint32_t C,
                                                      uint64_t *__restrict__ off, uint64_t *__restrict__ cb)
{
    __shared__ uint64_t s_off[16], s_cb[16];
    const uint64_t n = plan->n_allocs;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t carry_off = 0, carry_cb = 0;
    for (uint64_t base = 0; base < n; base += 1024) {
        const uint64_t k = base + threadIdx.x;
        const uint64_t sz = k < n ? size[k] : 0;
        const uint64_t e = round_up16(sz), c = (sz + C - 1) / C;
        const uint64_t ie = wave_incl_scan(e, lane), ic = wave_incl_scan(c, lane);
        if (lane == 63) {
            s_off[wave] = ie;
            s_cb[wave] = ic;
        }
        __syncthreads();
        uint64_t pre_off = carry_off, pre_cb = carry_cb, tot_off = 0, tot_cb = 0;
        for (int w = 0; w < 16; w++) {
            if (w < wave) {
                pre_off += s_off[w];
                pre_cb += s_cb[w];
            }
            tot_off += s_off[w];
            tot_cb += s_cb[w];
        }
        if (k < n) {
            off[k] = pre_off + ie - e;
            cb[k] = pre_cb + ic - c;
        }
        carry_off += tot_off;
        carry_cb += tot_cb;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        off[n] = carry_off;
        cb[n] = carry_cb;
        plan->data_bytes = carry_off;
        plan->n_chunks = carry_cb;
    }
}

// map[g] = k for every chunk g of row k: each wave takes 1024 chunks at a
// time, finds the first one's row by a binary search in cb and walks on (a
// wave per row left one wave with all chunks of one large allocation).
__global__ void k_chunk_map(const DevPlan *plan, const uint64_t *__restrict__ cb, uint32_t *__restrict__ map)
{
    const uint64_t n = plan->n_allocs;
    const int lane = threadIdx.x & 63;
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    const uint64_t N = n ? cb[n] : 0;
    constexpr uint64_t kStep = 1024;
    for (uint64_t g0 = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * kStep; g0 < N;
         g0 += waves * kStep) {
        const uint64_t g1 = g0 + kStep < N ? g0 + kStep : N;
        uint64_t lo = 0, hi = n;   // the last row with cb <= g0: cb[lo] <= g0 < cb[hi]
        while (hi - lo > 1) {
            const uint64_t mid = (lo + hi) / 2;
            if (cb[mid] <= g0)
                lo = mid;
            else
                hi = mid;
        }
        for (uint64_t k = lo, b = g0; b < g1; k++) {
            const uint64_t e = cb[k + 1] < g1 ? cb[k + 1] : g1;
            map_range(map, b + lane, e, 64, (uint32_t)k);
            b = b > e ? b : e;
        }
    }
}

// -------------------------------------------- K3/K4/K8: the chunk kernels
//
// Persistent workgroups take tiles of kTile chunk items from a counter; each tile's
// descriptors are staged in LDS once, then groups of waves_per_chunk waves
// take one item each.
//   kModePack:    read the allocation, write the dense image, CRC + flags.
//   kModeHash:    read the allocation, CRC + flags (incremental checkpoints).
//   kModeRestore: read the serialized chunk from staging (or zeros for a
//                 ZERO chunk), write the destination (exactly len bytes),
//                 recompute the CRC and compare with the stored one.

// Chunks per descriptor tile of the one-wave forms: few, so that the grid's
// window of memory stays narrow (random 4 KiB chunks: 128 per tile 1.64 ms for
// 4 GiB, 64 1.52, 32 1.51; the 1.6 GB batch 635 / 612 / 602 us).
constexpr int kTile = 32;
// Of chunks of at most 2 KiB: as many bytes per tile, since a tile's barrier and
// its chunks' latency cost the same whatever their size.  (512 MiB, tiles of 32
// / 64: random chunks of 1 KiB 0.357 / 0.309 ms, all ZERO 0.251 / 0.161, and
// 0.842 / 0.480 at 256 bytes; at 4 KiB both take the same.)
constexpr int kShortTile = 64;
constexpr int kRowsTile = 64;   // of the serving loop's launches

struct Desc {
    uint64_t src;   // pack/hash: source address; restore: staging address (0 for ZERO)
    uint64_t dst;   // pack: dense address; restore: destination address
    uint64_t g;     // chunk id
    uint32_t len;   // bytes in the chunk
    uint32_t zero;  // restore: the chunk is ZERO
    uint32_t want;  // the CRC to compare with (base for DIRTY, stored for restore),
                    // loaded with the descriptor so no wave waits on it at the end
    uint32_t has_base;  // pack/hash: a base chunk exists and want is its CRC
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <bool NT>
__device__ __forceinline__ uint4 ld16(const void *p)
{
    const Global<const u32x4> *q = (const Global<const u32x4> *)p;
    const u32x4 t = NT ? __builtin_nontemporal_load(q) : *q;
    return make_uint4(t.x, t.y, t.z, t.w);
}

template <bool NT>
__device__ __forceinline__ void st16(void *p, uint4 v)
{
    Global<u32x4> *q = (Global<u32x4> *)p;
    const u32x4 t = {v.x, v.y, v.z, v.w};
    if (NT)
        __builtin_nontemporal_store(t, q);
    else
        *q = t;
}

template <int MODE, bool NT>
__device__ __forceinline__ uint4 load_piece(const Desc &d, uint32_t start)
{
    if (MODE == kModeRestore) {
        if (d.zero)
            return make_uint4(0u, 0u, 0u, 0u);
        return ld16<NT>((const uint8_t *)d.src + start);   // staging pieces are padded to 16
    }
    // Allocations start on 16 bytes, and so do pieces: a tail's piece is loaded
    // whole (it lies in one page, so the load cannot fault) and the bytes past
    // the allocation are dropped.
    const uint4 v = ld16<NT>((const uint8_t *)d.src + start);
    return start + 16 <= d.len ? v : keep_bytes(v, d.len - start);
}

template <int MODE, bool NT>
__device__ __forceinline__ void store_piece(const Desc &d, uint32_t start, uint4 v)
{
    if (MODE == kModePack) {
        st16<NT>((uint8_t *)d.dst + start, v);            // dense image keeps the zero pad
    } else if (MODE == kModeRestore) {
        uint8_t *p = (uint8_t *)d.dst + start;
        if (start + 16 <= d.len)
            st16<NT>(p, v);
        else
            store_partial(p, d.len - start, v);
    }
}

// 16-byte loads each lane keeps in flight before hashing them.
constexpr int kLoadsInFlight = 4;

// Waits for the loads of v.  Called before the next loads are issued: on
// paths that issue a varying number of loads and then merge, a later wait for
// v could only be one for all of them.  (Hash-only, 4 GiB at 4 KiB chunks:
// 0.80 -> 0.705 ms, 6.1 TB/s.)
template <int B>
__device__ __forceinline__ void arrived(uint4 (&v)[B])
{
#pragma unroll
    for (int b = 0; b < B; b++)
        asm volatile("" : "+v"(v[b].x), "+v"(v[b].y), "+v"(v[b].z), "+v"(v[b].w));
}

// The register of the lane K places down (lane + K), for K < 16: a DPP row
// shift, with no LDS round trip.  Lanes whose source is outside their row of
// 16 get 0; the combine below reads only lanes whose source is inside.
template <int K>
__device__ __forceinline__ uint32_t dpp_down(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + K, 0xF, 0xF, true);
}

// Combine the 64 lanes' registers into lane 0: at level k, lane i (a multiple
// of 2^(k+1)) moves its register past the 16 * 2^k bytes of lane i + 2^k's
// share and adds that lane's register.  Levels 0-3 stay inside rows of 16
// lanes (DPP); levels 4 and 5 cross rows (__shfl_down).  The whole wave must
// be active.
static_assert(kTreeLevels == 6, "the combine is written out for 64 lanes");

__device__ __forceinline__ uint32_t wave_combine(const Tabs &T, uint32_t acc, int lane)
{
    uint32_t right = dpp_down<1>(acc);
    if ((lane & 1) == 0)
        acc = T.tree(0, acc) ^ right;
    right = dpp_down<2>(acc);
    if ((lane & 3) == 0)
        acc = T.tree(1, acc) ^ right;
    right = dpp_down<4>(acc);
    if ((lane & 7) == 0)
        acc = T.tree(2, acc) ^ right;
    right = dpp_down<8>(acc);
    if ((lane & 15) == 0)
        acc = T.tree(3, acc) ^ right;
    right = __shfl_down(acc, 16, 64);
    if ((lane & 31) == 0)
        acc = T.tree(4, acc) ^ right;
    right = __shfl_down(acc, 32, 64);
    if (lane == 0)
        acc = T.tree(5, acc) ^ right;
    return acc;
}

// The lane's register after one 16-byte piece, chained from register c.
__device__ __forceinline__ uint32_t chain_piece(const Tabs &T, uint32_t c, const uint4 &v)
{
    c = T.chain(c, v.x);
    c = T.chain(c, v.y);
    c = T.chain(c, v.z);
    return T.chain(c, v.w);
}

// The registers after the first B pieces of v, each chained from zero.  The chains go
// in lockstep, so that 2 B lookups are in flight; left to the scheduler, the
// larger kernels hashed piece by piece with two in flight (hash-only at 64 KiB
// chunks: 1.42 -> 1.53 ms).
template <int B>
__device__ __forceinline__ void chain_pieces(const Tabs &T, const uint4 (&v)[kLoadsInFlight],
                                             uint32_t (&c)[kLoadsInFlight])
{
#pragma unroll
    for (int b = 0; b < B; b++)
        c[b] = 0;
#pragma unroll
    for (int w = 0; w < 4; w++) {
#pragma unroll
        for (int b = 0; b < B; b++)
            c[b] ^= w == 0 ? v[b].x : w == 1 ? v[b].y : w == 2 ? v[b].z : v[b].w;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            uint32_t t0[B], t1[B];
#pragma unroll
            for (int b = 0; b < B; b++)
                T.chain_lookups(c[b], &t0[b], &t1[b]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < B; b++)
                c[b] = t0[b] ^ t1[b] ^ (c[b] >> 16);
        }
    }
}

constexpr int kPerRound = 64;   // 16-byte pieces per round (one per lane)

// One wave's share of a chunk: rounds [r_begin, r_end) of a window of r_win
// rounds of 1 KiB.  Returns the raw register of those rounds in lane 0 (as a
// message ending with the wave's last round) and ORs the data words into
// *orv.
template <int MODE, bool NT>
__device__ __forceinline__ uint32_t wave_rounds(const Tabs &T, const Desc &d, int lane, uint32_t r_begin,
                                                uint32_t r_end, uint32_t r_win, uint32_t *orv)
{
    constexpr int B = kLoadsInFlight;                                     // rounds per batch
    const uint32_t np = (d.len + 15) >> 4;                                // data pieces
    const uint32_t z = r_win * kPerRound - np;                            // leading zero pieces
    if (d.len == r_win * kPerRound * 16 && (MODE != kModeRestore || !d.zero)) {
        // The chunk fills the window exactly (uniform over the wave): every
        // piece is 16 bytes of data at offset (r * 64 + lane) * 16 and only
        // piece 0 carries the complemented init.
        uint32_t acc = 0, o = 0;
        for (uint32_t rb = r_begin; rb < r_end; rb += B) {
            uint4 v[B];
#pragma unroll
            for (int b = 0; b < B; b++)
                v[b] = rb + b < r_end ? ld16<NT>((const uint8_t *)d.src + ((rb + b) * kPerRound + lane) * 16)
                                      : make_uint4(0u, 0u, 0u, 0u);
            uint32_t c[B];
#pragma unroll
            for (int b = 0; b < B; b++) {
                const uint32_t r = rb + b;
                if (MODE != kModeHash && r < r_end)
                    st16<NT>((uint8_t *)d.dst + (r * kPerRound + lane) * 16, v[b]);
                o |= v[b].x | v[b].y | v[b].z | v[b].w;
                if (r == 0 && lane == 0)
                    v[b].x = ~v[b].x;
            }
            chain_pieces<B>(T, v, c);
#pragma unroll
            for (int b = 0; b < B; b++) {
                const uint32_t r = rb + b;
                if (r < r_end)
                    acc = (r > r_begin ? T.gap(acc) : 0u) ^ c[b];
            }
        }
        acc = wave_combine(T, acc, lane);
        *orv = o;
        return acc;
    }
    const uint32_t r0 = max(r_begin, z / kPerRound);                      // earlier rounds: all zero
    uint32_t acc = 0, o = 0;
    for (uint32_t rb = r0; rb < r_end; rb += B) {
        uint4 v[B];
#pragma unroll
        for (int b = 0; b < B; b++) {
            const int p = (int)((rb + b) * kPerRound + lane) - (int)z;
            v[b] = make_uint4(0u, 0u, 0u, 0u);
            if (rb + b < r_end && p >= 0)
                v[b] = load_piece<MODE, NT>(d, (uint32_t)p * 16);
        }
        // Each round's contribution is chained from a zero register, so the
        // rounds' lookups are independent; they are combined by Horner's rule
        // with the one-round shift.  Pieces past r_end are zero and add nothing.
        uint32_t c[B];
#pragma unroll
        for (int b = 0; b < B; b++) {
            const uint32_t r = rb + b;
            const int p = (int)(r * kPerRound + lane) - (int)z;
            if (r < r_end && p >= 0)
                store_piece<MODE, NT>(d, (uint32_t)p * 16, v[b]);
            o |= v[b].x | v[b].y | v[b].z | v[b].w;
            if (p == 0)
                v[b].x ^= init_mask(d.len);
        }
        chain_pieces<B>(T, v, c);
#pragma unroll
        for (int b = 0; b < B; b++) {
            const uint32_t r = rb + b;
            if (r < r_end)
                acc = (r > r0 ? T.gap(acc) : 0u) ^ c[b];
        }
    }
    acc = wave_combine(T, acc, lane);
    *orv = o;
    return acc;
}

// Chunks of at most one batch of rounds (r_win <= kLoadsInFlight, one wave
// per chunk): the same steps as wave_rounds, split into the loads and the
// rest, so that a wave can have the next chunk's loads in flight while it
// hashes, combines and finishes the current one.  The chunk sits at the end
// of the window, so of its rounds only the first has pieces before it (lanes
// below `skip`) and only the last a piece that its end cuts (lane 63); rounds
// of the window before the chunk are not touched.  All of this is uniform over
// the wave.
struct SmallItem {
    const uint8_t *src;
    uint8_t *dst;
    uint32_t len;
    uint32_t rounds;   // 1 .. kLoadsInFlight
    uint32_t skip;     // lanes of the first round before the chunk
    uint32_t tail;     // bytes of the last piece, when its end cuts it; else 0
    bool zero;         // restore: the chunk is ZERO
};

template <int MODE>
__device__ __forceinline__ SmallItem small_item(const Desc &d)
{
    SmallItem x;
    x.src = (const uint8_t *)uniform_u64(d.src);
    x.dst = MODE == kModeHash ? nullptr : (uint8_t *)uniform_u64(d.dst);
    x.len = uniform_u32(d.len);
    const uint32_t np = (x.len + 15) >> 4;
    x.rounds = (np + kPerRound - 1) / kPerRound;
    x.skip = x.rounds * kPerRound - np;
    x.tail = x.len & 15;
    x.zero = MODE == kModeRestore && uniform_u32(d.zero) != 0;
    return x;
}

// Byte offset of the lane's piece of round 0 (negative in skipped lanes).
__device__ __forceinline__ int small_offset(const SmallItem &x, int lane) { return (lane - (int)x.skip) * 16; }

template <int MODE, bool NT>
__device__ __forceinline__ void small_loads(const SmallItem &x, int lane, uint4 (&v)[kLoadsInFlight])
{
    const int o = small_offset(x, lane);
#pragma unroll
    for (int b = 0; b < kLoadsInFlight; b++) {
        v[b] = make_uint4(0u, 0u, 0u, 0u);
        if ((uint32_t)b < x.rounds && !(MODE == kModeRestore && x.zero) && (b > 0 || o >= 0)) {
            v[b] = ld16<NT>(x.src + (uint32_t)(o + b * kRoundBytes));
        }
    }
}

// An allocation's last piece is cut by its end (see load_piece); staging
// pieces are padded.  Not done where the piece is loaded: that would wait for it.
__device__ __forceinline__ void small_cut(const SmallItem &x, int lane, uint4 (&v)[kLoadsInFlight])
{
    if (x.tail == 0)
        return;
#pragma unroll
    for (int b = 0; b < kLoadsInFlight; b++)
        if ((uint32_t)b + 1 == x.rounds && lane == 63)
            v[b] = keep_bytes(v[b], x.tail);
}

// store: write the chunk's pieces (pack); a ZERO chunk's pieces are not
// stored, since the dense image leaves ZERO chunks unwritten.  Returns the raw
// register in lane 0.
template <int MODE, bool NT>
__device__ __forceinline__ uint32_t small_rest(const Tabs &T, const SmallItem &x, int lane,
                                               uint4 (&v)[kLoadsInFlight], bool store)
{
    constexpr int B = kLoadsInFlight;
    const int o = small_offset(x, lane);
    if (MODE != kModeHash && store) {
#pragma unroll
        for (int b = 0; b < B; b++)
            if ((uint32_t)b < x.rounds && (b > 0 || o >= 0)) {
                uint8_t *q = x.dst + (uint32_t)(o + b * kRoundBytes);
                if (MODE == kModeRestore && x.tail && (uint32_t)b + 1 == x.rounds && lane == 63)
                    store_partial(q, x.tail, v[b]);
                else
                    st16<NT>(q, v[b]);   // the dense image keeps the zero pad
            }
    }
    if (o == 0)   // the first data piece carries the complemented init
        v[0].x ^= init_mask(x.len);
    uint32_t c[B] = {};
    if (x.rounds > 2)
        chain_pieces<B>(T, v, c);
    else if (x.rounds == 2)
        chain_pieces<2>(T, v, c);
    else
        chain_pieces<1>(T, v, c);
    uint32_t acc = c[0];
#pragma unroll
    for (int b = 1; b < B; b++)
        if ((uint32_t)b < x.rounds)
            acc = T.gap(acc) ^ c[b];
    return wave_combine(T, acc, lane);
}

// Restore of a full-length ZERO chunk: its bytes are zeros, so its CRC is the
// CRC of C zero bytes, known beforehand; the wave stores the zeros and the
// stored CRC is compared with that value, with no table lookups.
template <bool NT>
__device__ __forceinline__ void restore_zero_chunk(const ChunkArgs &a, const Desc &d, int lane)
{
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
    for (uint32_t p = (uint32_t)lane * 16; p < d.len; p += 64 * 16)
        st16<NT>((uint8_t *)d.dst + p, zero);
    if (lane == 0 && a.zero_crc != d.want) {
        a.bad[d.g] = 1;
        atomicAdd(&a.plan_rw->bad_count, 1ull);
    }
}

// Pack and hash: a tile's CRCs and flags collect in LDS and go out together
// when the tile is done (k_chunks), to the device arrays and, when the plan
// has addresses there, straight into the image's pinned host memory: no
// copies after the pass (193 us of copies and 40 us of gaps for 2^21 chunks).
// A wave's later loads wait for its older stores, and one over the host link
// takes microseconds, so the host's share goes out for kOutResults chunks at
// a time: tile by tile it cost what the copies had (pack 2.30 -> 2.55 ms).
constexpr int kOutResults = 1024;

struct TileOut {
    Local<uint32_t> *crc;    // of the tile's slots
    Local<uint8_t> *flags;
};

// Pack / hash of a full-length ZERO chunk: its CRC is that of C zero bytes,
// known beforehand.
__device__ __forceinline__ void record_zero_chunk(const ChunkArgs &a, const TileOut &out, int slot, const Desc &d)
{
    uint8_t f = kFlagZero;
    if (!d.has_base || d.want != a.zero_crc)
        f |= kFlagDirty;
    out.crc[slot] = a.zero_crc;
    out.flags[slot] = f;
}

// crc: the CRC of the chunk at `slot` of the tile; called by one lane per chunk.
template <int MODE>
__device__ __forceinline__ void finish_chunk(const ChunkArgs &a, const TileOut &out, int slot, const Desc &d,
                                             uint32_t crc, bool nonzero)
{
    if (MODE == kModeRestore) {
        if (crc != d.want) {
            a.bad[d.g] = 1;
            atomicAdd(&a.plan_rw->bad_count, 1ull);
        }
    } else {
        uint8_t f = nonzero ? 0 : kFlagZero;
        if (!d.has_base || d.want != crc)
            f |= kFlagDirty;
        out.crc[slot] = crc;
        out.flags[slot] = f;
    }
}

// One chunk of the one-wave form, its loads in v: a full-length ZERO chunk
// of a restore is written as zeros; in a pack or hash, ZERO is known once the
// loads are in, so a ZERO chunk is not stored and a full-length one not
// hashed; every other chunk is hashed (and stored) and finished.
template <int MODE, bool NT>
__device__ __forceinline__ void small_chunk(const ChunkArgs &a, const Tabs &T, const TileOut &out, int slot,
                                            const Desc &d, const SmallItem &x, int lane, uint32_t C,
                                            uint4 (&v)[kLoadsInFlight])
{
    if (MODE == kModeRestore && x.zero && x.len == C) {
        restore_zero_chunk<NT>(a, d, lane);
        return;
    }
    bool nonzero = true;
    if (MODE != kModeRestore) {
        small_cut(x, lane, v);
        uint32_t o = 0;
#pragma unroll
        for (int b = 0; b < kLoadsInFlight; b++)
            o |= v[b].x | v[b].y | v[b].z | v[b].w;
        nonzero = __ballot(o != 0) != 0;   // uniform over the wave
        if (!nonzero && x.len == C) {
            if (lane == 0)
                record_zero_chunk(a, out, slot, d);
            return;
        }
    }
    const uint32_t raw = small_rest<MODE, NT>(T, x, lane, v, nonzero);
    const uint32_t crc = finish_crc(T, uniform_u32(raw), x.len, lane);
    if (lane == 0)
        finish_chunk<MODE>(a, out, slot, d, crc, nonzero);
}

// ------------------------------- long form (one wave per chunk, C > 4 KiB)
//
// The wave goes through its chunks batch by batch (kLoadsInFlight rounds), in
// the window of wave_rounds, with the next batch's loads (of this chunk or of
// the wave's next) in flight while it hashes and stores the current one.
// Bound by HBM.  Every byte of a pack is stored (unlike in the small form, a
// ZERO chunk's too: callers find zeros there), but until a chunk's first
// non-zero batch nothing is hashed.  If one comes, the zeros' part of the
// register is the complemented init moved over them.  A full-length ZERO chunk
// has a known CRC.  (4 GiB in chunks of 64 KiB, random bytes or half of the
// allocations zero: 1.64 ms, 5.2 TB/s read and written; with the zeros left
// unwritten, which callers that use a buffer again saw, 1.18.)

// One chunk as the wave sees it: uniform over the wave.
struct LongItem {
    uint64_t src, dst;   // (of a ZERO chunk both the destination)
    uint32_t len;
    uint32_t z;       // leading zero pieces of the window
    uint32_t r0;      // first round with data
    bool zero;        // restore: the chunk is ZERO
    bool skip;        // restore: ZERO and full-length, written without hashing
};

template <int MODE>
__device__ __forceinline__ LongItem long_item(const Desc &d, uint32_t r_win, uint32_t C)
{
    LongItem x;
    x.src = uniform_u64(d.src);
    x.dst = MODE == kModeHash ? 0 : uniform_u64(d.dst);
    x.len = uniform_u32(d.len);
    x.z = r_win * kPerRound - ((x.len + 15) >> 4);
    x.r0 = x.z / kPerRound;
    x.zero = MODE == kModeRestore && uniform_u32(d.zero) != 0;
    x.skip = MODE == kModeRestore && x.zero && x.len == C;
    if (x.skip)
        x.r0 = r_win - 1;   // one batch
    if (MODE == kModeRestore && x.zero)
        x.src = x.dst;      // see long_loads
    return x;
}

// The lane's piece of the chunk in round r (negative before the chunk).
__device__ __forceinline__ int long_piece(const LongItem &x, int lane, uint32_t r)
{
    return (int)(r * kPerRound + lane) - (int)x.z;
}

// Whether every lane has a piece of the chunk in each round of the batch at rb.
__device__ __forceinline__ bool long_full(const LongItem &x, uint32_t r_win, uint32_t rb)
{
    return rb * kPerRound >= x.z && rb + kLoadsInFlight <= r_win;
}

// The same loads in every case, of the chunk's first or last piece where the
// lane has none and of the destination for a ZERO chunk: with loads in one or
// both arms of a branch, registers were copied (and so waited for) where the
// arms met.  (Hash-only, 8 GiB at 64 KiB chunks: 1.35 -> 1.31 ms, 6.5 TB/s.)
template <int MODE, bool NT>
__device__ __forceinline__ void long_loads(const LongItem &x, int lane, uint32_t r_win, uint32_t rb,
                                           uint4 (&v)[kLoadsInFlight])
{
    int p[kLoadsInFlight];
#pragma unroll
    for (int b = 0; b < kLoadsInFlight; b++)
        p[b] = long_piece(x, lane, rb + b);
    if (!long_full(x, r_win, rb)) {
        const int end = (int)((x.len - 1) >> 4);
#pragma unroll
        for (int b = 0; b < kLoadsInFlight; b++)
            p[b] = min(max(p[b], 0), end);
    }
#pragma unroll
    for (int b = 0; b < kLoadsInFlight; b++)
        v[b] = ld16<NT>((const uint8_t *)x.src + (uint32_t)p[b] * 16);
}

// What the loads brought that is not the chunk's, zeroed: lanes without a
// piece, and the bytes after an allocation's end (see load_piece; staging
// pieces are padded).
template <int MODE>
__device__ __forceinline__ void long_cut(const LongItem &x, int lane, uint32_t r_win, uint32_t rb,
                                         uint4 (&v)[kLoadsInFlight])
{
    if (!long_full(x, r_win, rb) || (MODE == kModeRestore && x.zero)) {
#pragma unroll
        for (int b = 0; b < kLoadsInFlight; b++)
            if (rb + b >= r_win || long_piece(x, lane, rb + b) < 0 || (MODE == kModeRestore && x.zero))
                v[b] = make_uint4(0u, 0u, 0u, 0u);
    }
    if (MODE != kModeRestore && (x.len & 15) != 0 && rb + kLoadsInFlight >= r_win) {
#pragma unroll
        for (int b = 0; b < kLoadsInFlight; b++)
            if (rb + b + 1 == r_win && lane == 63)
                v[b] = keep_bytes(v[b], x.len & 15);
    }
}

template <int MODE, bool NT>
__device__ __forceinline__ void long_store(const LongItem &x, int p, uint4 v)
{
    uint8_t *q = (uint8_t *)x.dst + (uint32_t)p * 16;
    if (MODE == kModePack || (uint32_t)p * 16 + 16 <= x.len)
        st16<NT>(q, v);   // the dense image keeps the zero pad
    else
        store_partial(q, x.len - (uint32_t)p * 16, v);
}

// The register after the zero rounds [r0, r): the complemented init of the
// first piece, in the lane that holds it, moved over the rest.
__device__ __forceinline__ uint32_t long_zero_prefix(const Tabs &T, const LongItem &x, int lane, uint32_t r)
{
    uint4 first = make_uint4((uint32_t)lane == x.z % kPerRound ? init_mask(x.len) : 0u, 0u, 0u, 0u);
    uint32_t acc = chain_piece(T, 0u, first);
    for (uint32_t k = x.r0 + 1; k < r; k++)
        acc = T.gap(acc);
    return acc;
}

// One batch of a chunk: stored, hashed into *acc; after the last batch the
// chunk is finished.  *seen: a non-zero batch has come (pack and hash).
template <int MODE, bool NT>
__device__ __forceinline__ void long_batch(const ChunkArgs &a, const Tabs &T, const TileOut &out, int slot,
                                           const Desc &d, const LongItem &x, int lane, uint32_t r_win, uint32_t rb,
                                           uint4 (&v)[kLoadsInFlight], uint32_t *acc, bool *seen)
{
    constexpr int B = kLoadsInFlight;
    const bool last = rb + B >= r_win;
    if (MODE == kModeRestore && x.skip) {
        restore_zero_chunk<NT>(a, d, lane);
        return;
    }
    long_cut<MODE>(x, lane, r_win, rb, v);
    if (MODE != kModeHash) {
        if (long_full(x, r_win, rb) && !(MODE == kModeRestore && last && (x.len & 15) != 0)) {
            uint8_t *q = (uint8_t *)x.dst + (uint32_t)long_piece(x, lane, rb) * 16;
#pragma unroll
            for (int b = 0; b < B; b++)
                st16<NT>(q + b * kRoundBytes, v[b]);
        } else {
#pragma unroll
            for (int b = 0; b < B; b++) {
                const int p = long_piece(x, lane, rb + b);
                if (rb + b < r_win && p >= 0)
                    long_store<MODE, NT>(x, p, v[b]);
            }
        }
    }
    if (MODE != kModeRestore && !*seen) {
        uint32_t o = 0;
#pragma unroll
        for (int b = 0; b < B; b++)
            o |= v[b].x | v[b].y | v[b].z | v[b].w;
        if (__ballot(o != 0) == 0) {
            if (!last)
                return;
            if (x.len == a.C) {
                if (lane == 0)
                    record_zero_chunk(a, out, slot, d);
                return;
            }
            // a short ZERO chunk: its CRC from the init alone
            const uint32_t raw = wave_combine(T, long_zero_prefix(T, x, lane, r_win), lane);
            const uint32_t crc = finish_crc(T, uniform_u32(raw), x.len, lane);
            if (lane == 0)
                finish_chunk<MODE>(a, out, slot, d, crc, false);
            return;
        }
        *seen = true;
        if (rb > x.r0)
            *acc = long_zero_prefix(T, x, lane, rb);
    }
    uint32_t c[B];
    uint32_t s = *acc;
    if (rb == x.r0 && long_piece(x, lane, rb) == 0)   // the first data piece carries the complemented init
        v[0].x ^= init_mask(x.len);
    chain_pieces<B>(T, v, c);
#pragma unroll
    for (int b = 0; b < B; b++)
        if (rb + b < r_win)
            s = T.gap(s) ^ c[b];   // a zero register stays zero: no case for the first round
    *acc = s;
    if (last) {
        const uint32_t crc = finish_crc(T, uniform_u32(wave_combine(T, s, lane)), x.len, lane);
        if (lane == 0)
            finish_chunk<MODE>(a, out, slot, d, crc, true);
    }
}

// The chunk of item i: i, or ids[i] in a delta restore.
template <int MODE>
__device__ __forceinline__ uint64_t item_chunk(const ChunkArgs &a, uint64_t i)
{
    if (MODE == kModeRestore)
        i += a.item_begin;
    return (MODE == kModeRestore && a.ids) ? a.ids[i] : i;
}

// A row of the allocation table with its place in the layout.
struct AllocRow {
    uint64_t addr;   // restore: of the destination
    uint64_t size, off, cb;
};

template <int MODE>
__device__ __forceinline__ AllocRow alloc_row(const ChunkArgs &a, uint32_t k)
{
    return {MODE == kModeRestore ? a.dst[k] : a.src[k], a.size[k], MODE == kModePack ? a.off[k] : 0, a.cb[k]};
}

// The descriptor of item i, chunk g of allocation row k.
template <int MODE>
__device__ __forceinline__ Desc make_desc(const ChunkArgs &a, uint64_t i, uint64_t g, uint32_t k, const AllocRow &row,
                                          uint32_t C)
{
    if (MODE == kModeRestore)
        i += a.item_begin;
    const uint64_t start = (g - row.cb) * C;
    const uint64_t rest = row.size - start;
    Desc d;   // only what the mode reads is set: the rest takes no registers
    d.len = (uint32_t)(rest < C ? rest : C);
    if (MODE == kModeRestore) {
        d.g = g;
        d.zero = a.want_flags[g] & kFlagZero;
        d.want = a.want_crc[g];
        d.src = d.zero ? 0 : (uint64_t)(a.staging + (a.soff[i] - a.soff_base));
        d.dst = row.addr + start;
    } else {
        // the base chunk: the same id when the base has this table, else the
        // same chunk of the base allocation with this allocation's id
        uint64_t bg = g;
        d.has_base = a.base_crc != nullptr;
        if (a.base_cb) {
            const uint64_t b0 = a.base_cb[k];
            d.has_base = b0 != kNoBase;
            bg = b0 + (g - row.cb);
        }
        d.want = d.has_base ? a.base_crc[bg] : 0;
        d.src = row.addr + start;
        if (MODE == kModePack)
            d.dst = (uint64_t)(a.dense + row.off + start);
    }
    return d;
}

// --------------------------------------------- quad form (hash only, C <= 4 KiB)
//
// Each row of 16 lanes hashes a chunk of its own, four chunks per wave.  A
// chunk of len bytes sits at the end of a window of r_win rounds of 1 KiB as
// in the one-wave form.  The window is cut into stretches of 256 bytes, one
// 16-byte piece per lane: lane l of the row reads piece l of every stretch,
// so each load instruction covers 256 contiguous bytes per row.  The lane
// chains its pieces in order into one register; the last word of a piece
// (but the last piece's) uses the skip operator, which also moves the
// register over the other 15 lanes' pieces of the stretch, so no separate
// round operator is needed.  The row's 16 registers are then combined inside
// the row with the tree operators for 16, 32, 64 and 128 bytes.  The
// cross-lane tree, the flag test and the finish are shared by four chunks,
// which is what this form saves over one wave per chunk.
constexpr int kQuadRows = 64 / kQuadLanes;        // chunks per wave
constexpr int kQuadPieces = 4;                    // 16-byte pieces per lane per round
constexpr int kQuadRoundPieces = kQuadLanes * kQuadPieces;
constexpr int kQuadMaxRounds = 4;
static_assert(kQuadRoundPieces * 16 == kRoundBytes, "a row round is one wave round long");
static_assert(kQuadRows == 4, "the row flags are 16-bit fields of the wave ballot");

// descriptor tile of the quad form: four chunks per wave and four quads per
// wave of a 1024-thread workgroup between two barriers
constexpr int kQuadTile = 256;

// Loads of round b of a row's window (b < r_win): piece j of the lane is
// window piece (4 b + j) * 16 + lr.
template <bool NT>
__device__ __forceinline__ void quad_loads(const Desc &d, bool valid, bool exact, int lr, uint32_t r_win, uint32_t b,
                                           uint4 (&v)[kQuadPieces])
{
    const uint32_t first = b * kQuadRoundPieces + lr;   // window piece of v[0]
    if (exact) {   // every row's chunk fills its window: whole pieces, no offset
#pragma unroll
        for (int j = 0; j < kQuadPieces; j++)
            v[j] = ld16<NT>((const uint8_t *)d.src + (first + j * kQuadLanes) * 16);
        return;
    }
    const int z = valid ? (int)(r_win * kQuadRoundPieces) - (int)((d.len + 15) >> 4) : 0;
#pragma unroll
    for (int j = 0; j < kQuadPieces; j++) {
        const int p = (int)(first + j * kQuadLanes) - z;
        v[j] = make_uint4(0u, 0u, 0u, 0u);
        if (valid && p >= 0)
            v[j] = load_piece<kModeHash, NT>(d, (uint32_t)p * 16);
    }
}

// Chains round b's pieces into the lane's register (T is the quad table set:
// its gap operator is the skip) and ORs their data words into *o.
__device__ __forceinline__ void quad_hash(const Tabs &T, const Desc &d, bool valid, bool exact, int lr,
                                          uint32_t r_win, uint32_t b, uint4 (&v)[kQuadPieces], uint32_t *acc,
                                          uint32_t *o)
{
    const uint32_t first = b * kQuadRoundPieces + lr;
    const int z = (valid && !exact) ? (int)(r_win * kQuadRoundPieces) - (int)((d.len + 15) >> 4) : 0;
    const bool last_round = b + 1 == r_win;   // uniform over the wave
    uint32_t r = *acc;
#pragma unroll
    for (int j = 0; j < kQuadPieces; j++) {
        *o |= v[j].x | v[j].y | v[j].z | v[j].w;
        // the first data byte's piece carries the complemented init (zero
        // pieces before it leave the register at zero)
        if (exact) {
            if (first + j * kQuadLanes == 0)
                v[j].x = ~v[j].x;
        } else if (valid && (int)(first + j * kQuadLanes) == z) {
            v[j].x ^= init_mask(d.len);
        }
        r = T.chain(r, v[j].x);
        r = T.chain(r, v[j].y);
        r = T.chain(r, v[j].z);
        if (j == kQuadPieces - 1 && last_round)
            r = T.chain(r, v[j].w);   // the window ends with this stretch
        else
            r = T.gap(r ^ v[j].w);    // 4 bytes, then the other lanes' pieces
    }
    *acc = r;
}

// The row's 16 registers combined into the row's lane 0 (DPP row shifts):
// at level k, lane i moves its register past the 16 << k bytes of lane
// i + 2^k's pieces and adds that lane's register.
__device__ __forceinline__ uint32_t quad_combine(const Tabs &T, uint32_t acc, int lane)
{
    uint32_t right = dpp_down<1>(acc);
    if ((lane & 1) == 0)
        acc = T.tree(0, acc) ^ right;
    right = dpp_down<2>(acc);
    if ((lane & 3) == 0)
        acc = T.tree(1, acc) ^ right;
    right = dpp_down<4>(acc);
    if ((lane & 7) == 0)
        acc = T.tree(2, acc) ^ right;
    right = dpp_down<8>(acc);
    if ((lane & 15) == 0)
        acc = T.tree(3, acc) ^ right;
    return acc;
}

// Tile counters: every taker (a workgroup of a chunk launch, a wave of a
// gather) takes tiles until its first miss (a value of at least n_tiles), so
// a launch makes n_tiles + takers takes.  The taker whose miss is the last
// take of the launch sets the counter back to zero for the next launch on the
// same plan (such launches are stream-ordered, and the host writes every plan
// with zero counters).
__device__ __forceinline__ uint64_t take_tile(unsigned long long *ctr)
{
    return atomicAdd(ctr, 1ull);
}

// A selection tile's total (K5): bytes in the low 48 bits, count above.
__device__ __forceinline__ uint64_t sel_pack(uint64_t bytes, uint64_t count) { return (count << 48) | bytes; }
__device__ __forceinline__ uint64_t sel_bytes(uint64_t v) { return v & ((1ull << 48) - 1); }
__device__ __forceinline__ uint64_t sel_count(uint64_t v) { return v >> 48; }

// What a chunk's flags say: whether its bytes are selected, whether its id is.
__device__ __forceinline__ void sel_flags(int mode, uint8_t f, bool *take, bool *id)
{
    *take = !(f & kFlagZero) && (mode == kSelDirtyNonZero ? (f & kFlagDirty) != 0 : mode != kSelBad);
    *id = mode == kSelDirtyNonZero ? (f & kFlagDirty) != 0 : mode == kSelBad && f != 0;
}

// Sum over the wave, in every lane.
__device__ __forceinline__ uint64_t wave_sum(uint64_t v)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1)
        v += __shfl_xor(v, d, 64);
    return v;
}

// The next chunk of the workgroup's tile, for one wave.
__device__ __forceinline__ int take_chunk(int *next, int lane)
{
    int v = 0;
    if (lane == 0)
        v = atomicAdd(next, 1);
    return __builtin_amdgcn_readfirstlane(v);
}

__device__ __forceinline__ void tiles_done(unsigned long long *ctr, uint64_t miss, uint64_t n_tiles, uint64_t takers)
{
    if (miss == n_tiles + takers - 1)
        atomicExch(ctr, 0ull);
}

// FORM: kFormWave (several waves per chunk), kFormLong (one wave per chunk,
// above), kFormSmall (every chunk is one batch of rounds and one wave hashes
// it; the wave keeps the next chunk's loads in flight while it finishes the
// current one) or kFormQuad (above).  The host picks the form that applies.
constexpr int kFormWave = 0;
constexpr int kFormSmall = 1;
constexpr int kFormQuad = 2;
constexpr int kFormLong = 3;

// v, opaque to the optimizer where it is used: what is computed from it once
// per tile stays there.  Otherwise the lanes' addresses into every array are
// kept in registers across the hash loops, which then have fewer lookups in
// flight (hash-only at 64 KiB chunks: 1.43 -> 1.56 ms).
__device__ __forceinline__ uint32_t per_tile(uint32_t v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// The operator tables into LDS, eight 16-byte loads per thread in flight (in
// 4-byte steps the staging took half of a small launch).  `between` runs
// with the first loads in flight.
static_assert(kRepWords % 4 == 0, "staged in 16-byte pieces");

template <class F>
__device__ __forceinline__ void stage_tables(uint32_t *tabs, const uint32_t *__restrict__ src, F between)
{
    constexpr int n = kRepWords / 4;
    constexpr int B = 8;
    const uint4 *s = (const uint4 *)src;
    uint4 *d = (uint4 *)tabs;
    bool first = true;
    for (int base = threadIdx.x; base < n; base += B * blockDim.x) {
        uint4 v[B];
#pragma unroll
        for (int b = 0; b < B; b++) {
            const int i = base + b * (int)blockDim.x;
            v[b] = s[i < n ? i : n - 1];
        }
        if (first)   // every thread has a first iteration
            between();
        first = false;
#pragma unroll
        for (int b = 0; b < B; b++)
            if (base + b * (int)blockDim.x < n)
                d[base + b * blockDim.x] = v[b];
    }
}

// table: null, or a table of at most kRowTile rows from the launch's arguments
// (then a's row arrays and map are not used, and the launch has at most kTile
// chunks per workgroup, so that one tile each takes them all).
template <int MODE, bool NT, int FORM, bool TABLE>
__device__ __forceinline__ void chunks(const ChunkArgs &a, const SmallTable *table)
{
    __shared__ __attribute__((aligned(16))) uint32_t tabs[kRepWords];
    // two descriptor tiles: the first wave loads the next tile's descriptors
    // while the workgroup works on the current one
    constexpr int kDescTile = FORM == kFormQuad ? kQuadTile : FORM == kFormSmall ? kShortTile : kTile;
    __shared__ Desc desc[2][kDescTile];
    // results of the last 2 * kOutTiles tiles: a tile's go to the device arrays
    // when it is done, kOutTiles tiles' to the host at a time
    constexpr int kOutTile = MODE == kModeRestore ? 1 : kDescTile;
    constexpr int kOutTiles = MODE == kModeRestore ? 1 : kOutResults / (FORM == kFormSmall ? kTile : kDescTile);
    __shared__ __attribute__((aligned(16))) uint32_t s_crc[2 * kOutTiles][kOutTile];
    __shared__ __attribute__((aligned(16))) uint8_t s_flags[2 * kOutTiles][kOutTile];
    __shared__ uint64_t s_done[2 * kOutTiles];   // the tiles
    __shared__ uint32_t s_part[16];
    __shared__ uint32_t s_nz[16];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const Tabs T = make_tabs(tabs, lane);
    const int nwaves = blockDim.x >> 6;
    const int W = a.waves_per_chunk;
    const int groups = nwaves / W, group = wave / W, wig = wave % W;
    const uint32_t C = a.C;
    const uint32_t r_full = (C + kRoundBytes - 1) / kRoundBytes;
    const uint32_t rw = (r_full + W - 1) / W;            // rounds per wave
    const uint32_t r_win = rw * W;
    const uint64_t M = a.n_known ? a.n_known
                       : (MODE != kModeRestore) ? a.plan->n_chunks
                       : a.item_end ? a.item_end - a.item_begin : a.plan->n_items;

    // The items go in tiles: workgroup b's first tile is tile b, and the rest
    // are taken in order from a counter in the plan, one tile ahead (thread 0
    // takes the tile after the next while the workgroup works on the current
    // one), so the grid sweeps the memory in order and a workgroup whose tiles
    // are cheap (ZERO chunks, read only) takes more of them.
    // A tile holds at most kDescTile chunks (in the small form kTile of more
    // than 2 KiB) and, for large chunks, about 1 MiB (but at least one chunk per
    // group of waves), so that a launch has many tiles per workgroup and its
    // last tiles end close together; and few enough for two tiles per
    // workgroup, down to one chunk per group of waves: 2350 chunks in tiles of
    // 64 kept 37 of 256 workgroups busy.  (Four per workgroup: hash-only of
    // 131072 chunks 139 us, two 121, one 146.)
    int tile = kDescTile < (int)blockDim.x ? kDescTile : (int)blockDim.x;
    const int least = FORM == kFormQuad ? kQuadRows * nwaves : groups;
    if (FORM == kFormWave || FORM == kFormLong) {
        const int by_bytes = (int)((1u << 20) / C);
        const int want = by_bytes > groups ? by_bytes : groups;
        tile = want < tile ? want : tile;
    }
    if (FORM == kFormSmall && r_full > 2)
        tile = kTile < tile ? kTile : tile;
    int tile_log = 31 - __builtin_clz(tile);   // a power of two (as `least` is)
    while ((1 << tile_log) > least && ((uint64_t)2 * gridDim.x << tile_log) > M)
        tile_log--;
    if (TABLE)
        while (((uint64_t)gridDim.x << tile_log) < M)
            tile_log++;
    tile = 1 << tile_log;
    const uint64_t n_tiles = (M + tile - 1) / tile;
    if (blockIdx.x >= n_tiles)
        return;   // fewer tiles than workgroups: none is taken from the counter
    if (MODE == kModeRestore && a.plan->sel_bad)
        return;   // the flags do not match the serialized bytes: nothing is read or written
    const uint64_t n_dyn = n_tiles > gridDim.x ? n_tiles - gridDim.x : 0;   // tiles from the counter
    const bool stager = (int)threadIdx.x < tile;
    // A tile's first chunks are the waves' own; the rest go to whichever wave is
    // free next, so that ZERO chunks and a wave that waits for the host link
    // cost the others nothing.
    __shared__ int s_next[2];
    __shared__ uint64_t s_tile[2];
    uint64_t cur = blockIdx.x, nxt = n_tiles;    // the tile worked on, the tile staged meanwhile
    // The first descriptors' two dependent loads run beside the tables' (the
    // first goes out before them, the rest behind them).
    const uint64_t i0 = cur * tile + threadIdx.x;
    const bool have0 = stager && i0 < M;
    uint64_t g0_first = 0;
    uint32_t k0 = 0;
    if (have0) {
        g0_first = item_chunk<MODE>(a, i0);
        if (!TABLE)
            k0 = a.map[g0_first];
    }
    Desc d0;
    stage_tables(tabs, a.tables, [&]() {
        if constexpr (TABLE) {
            // Every stager is in the first wave (a tile has at most 64 chunks
            // here): it scans the rows, one per lane, and searches its chunks'
            // rows among its lanes.
            if (wave == 0) {
                AllocRow r;
                r.addr = table->addr[lane];
                r.size = table->size[lane];   // 0 past the last row
                const uint64_t e = round_up16(r.size), nc = (r.size + C - 1) / C;
                r.off = wave_incl_scan(e, lane) - e;
                r.cb = wave_incl_scan(nc, lane) - nc;
                for (uint32_t step = kRowTile / 2; step; step >>= 1)   // the last row with cb <= g
                    if (__shfl(r.cb, k0 + step, 64) <= g0_first)
                        k0 += step;
                r = {__shfl(r.addr, k0, 64), __shfl(r.size, k0, 64), __shfl(r.off, k0, 64), __shfl(r.cb, k0, 64)};
                if (have0)
                    d0 = make_desc<MODE>(a, i0, g0_first, k0, r, C);
            }
        } else if (have0) {
            d0 = make_desc<MODE>(a, i0, g0_first, k0, alloc_row<MODE>(a, k0), C);
        }
        if (threadIdx.x == 0 && n_dyn) {
            const uint64_t v = take_tile(&a.plan_rw->tile_next);
            if (v >= n_dyn)
                tiles_done(&a.plan_rw->tile_next, v, n_dyn, gridDim.x);
            nxt = gridDim.x + v;
        }
    });
    if (have0)
        desc[0][threadIdx.x] = d0;
    if (threadIdx.x == 0) {
        s_tile[0] = nxt;
        s_next[0] = 0;
    }
    __syncthreads();
    nxt = uniform_u64(s_tile[0]);
    int buf = 0;
    // The results of the tile before (iteration it - 1), then, when the host
    // takes them and a group of kOutTiles tiles is full or the last tile done,
    // of the group.
    const auto put_results = [&](uint32_t it, uint64_t done, int prev, bool end) {   // prev: its descriptors
        if (MODE == kModeRestore)
            return;
        const uint32_t row = (it - 1) % (2 * kOutTiles);
        const uint32_t tid = per_tile(threadIdx.x);
        const uint64_t g = done * tile + tid;
        const bool mine = tid < (uint32_t)tile && g < M;
        uint8_t f = 0;
        if (mine) {
            f = s_flags[row][tid];
            a.crc[g] = s_crc[row][tid];
            a.flags[g] = f;
        }
        if (a.sel_totals && 64 * wave < tile) {   // the selection's totals (uniform over the wave)
            bool take, id;
            sel_flags(MODE == kModeHash ? kSelDirtyNonZero : kSelNonZero, f, &take, &id);
            const uint64_t v = wave_sum(
                mine ? sel_pack(take ? round_up16(desc[prev][tid].len) : 0, id ? 1 : 0) : 0);
            if (lane == 0 && v)   // a tile (a power of two of at most 256 chunks) lies in one selection tile
                atomicAdd((unsigned long long *)&a.sel_totals[g / kSelTile], (unsigned long long)v);
        }
        if (!a.to_host || !(end || it % kOutTiles == 0))
            return;
        Global<uint32_t> *h_crc = (Global<uint32_t> *)a.plan->h_crc;
        Global<uint8_t> *h_flags = (Global<uint8_t> *)a.plan->h_flags;
        const uint32_t first = (it - 1) / kOutTiles * kOutTiles;   // iteration of the group's first tile
        // four chunks per lane: whole 16- and 4-byte stores over the link, by the
        // last wave (every wave in the quad form, whose quads are dealt out)
        const uint32_t step = FORM == kFormQuad ? blockDim.x : 64u;
        if (FORM != kFormQuad && wave != nwaves - 1)
            return;
        for (uint32_t i = 4 * (tid % step); i < (it - first) * tile; i += 4 * step) {
            const uint32_t r = (first + (i >> tile_log)) % (2 * kOutTiles), c = i & (tile - 1);
            const uint64_t h = s_done[r] * tile + c;
            if (tile >= 4 && h + 4 <= M) {
                *(Global<u32x4> *)(h_crc + h) = *(const u32x4 *)&s_crc[r][c];
                *(Global<uint32_t> *)(h_flags + h) = *(const uint32_t *)&s_flags[r][c];
            } else {
                for (uint32_t j = i; j < i + 4 && j < (it - first) * tile; j++) {
                    const uint32_t rj = (first + (j >> tile_log)) % (2 * kOutTiles), cj = j & (tile - 1);
                    const uint64_t hj = s_done[rj] * tile + cj;
                    if (hj < M) {
                        h_crc[hj] = s_crc[rj][cj];
                        h_flags[hj] = s_flags[rj][cj];
                    }
                }
            }
        }
    };
    uint64_t done = 0;
    uint32_t its = 0;
    for (uint32_t it = 0; cur < n_tiles; it++, buf ^= 1) {
        __syncthreads();   // tables, this tile's descriptors and the last take are in LDS
        if (it > 0)
            nxt = uniform_u64(s_tile[it & 1]);   // taken during the previous iteration
        if (threadIdx.x == 0)
            s_next[buf ^ 1] = 0;   // last used in the tile before the barrier
        uint64_t taken = n_dyn;
        if (threadIdx.x == 0 && nxt < n_tiles)
            taken = take_tile(&a.plan_rw->tile_next);   // its value is first needed at the end of the tile
        const uint64_t g0 = cur * tile, hi = g0 + tile < M ? g0 + tile : M;
        const uint64_t n0 = nxt * tile, n1 = nxt < n_tiles ? (n0 + tile < M ? n0 + tile : M) : n0;
        Desc nd;
        const uint32_t tid = per_tile(threadIdx.x);
        const bool have_nd = !TABLE && tid < (uint32_t)tile && n0 + tid < n1;
        if (have_nd) {   // loads in flight during the tile
            const uint64_t g = item_chunk<MODE>(a, n0 + tid);
            const uint32_t k = a.map[g];
            nd = make_desc<MODE>(a, n0 + tid, g, k, alloc_row<MODE>(a, k), C);
        }
        const int cnt = (int)(hi - g0);   // uniform over the workgroup, at most tile
        const uint32_t row = MODE == kModeRestore ? 0 : it % (2 * kOutTiles);
        const TileOut out = {(Local<uint32_t> *)s_crc[row], (Local<uint8_t> *)s_flags[row]};
        if (it > 0)
            put_results(it, done, buf ^ 1, false);   // complete since the barrier
        if constexpr (FORM == kFormQuad) {
            static_assert(MODE == kModeHash, "the quad form only hashes");
            // This wave's quads of the tile, round by round: the next round's
            // loads (of this quad, or the first of the next) are in flight
            // while the current round is hashed.
            const int q = lane / kQuadLanes, lr = lane & (kQuadLanes - 1);
            const int stride = kQuadRows * nwaves, first = kQuadRows * wave;
            const int nq = first < cnt ? (cnt - first + stride - 1) / stride : 0;   // uniform over the wave
            Desc dn;
            bool vn = false, en = false;
            uint4 cur[kQuadPieces], nxt[kQuadPieces];
            if (nq > 0) {
                vn = first + q < cnt;
                if (vn)
                    dn = desc[buf][first + q];
                en = __ballot(!vn || dn.len != r_win * kRoundBytes) == 0;
                quad_loads<NT>(dn, vn, en, lr, r_win, 0, nxt);
            }
            for (int k = 0; k < nq; k++) {
                const Desc dc = dn;
                const bool vc = vn, ec = en;
                uint32_t acc = 0, orv = 0;
                for (uint32_t b = 0; b < r_win; b++) {
#pragma unroll
                    for (int j = 0; j < kQuadPieces; j++)
                        cur[j] = nxt[j];
                    arrived(cur);
                    if (b + 1 < r_win) {
                        quad_loads<NT>(dc, vc, ec, lr, r_win, b + 1, nxt);
                    } else if (k + 1 < nq) {
                        const int t = first + (k + 1) * stride + q;
                        vn = t < cnt;
                        if (vn)
                            dn = desc[buf][t];
                        en = __ballot(!vn || dn.len != r_win * kRoundBytes) == 0;
                        quad_loads<NT>(dn, vn, en, lr, r_win, 0, nxt);
                    }
                    quad_hash(T, dc, vc, ec, lr, r_win, b, cur, &acc, &orv);
                }
                const uint32_t raw = quad_combine(T, acc, lane);
                const uint64_t nz = __ballot(orv != 0);
                const uint32_t crc = finish_crc(T, __shfl(raw, lane & ~(kQuadLanes - 1), 64), vc ? dc.len : 16u, lane);
                if (vc && lr == 0)
                    finish_chunk<MODE>(a, out, first + k * stride + q, dc, crc,
                                       ((nz >> (q * kQuadLanes)) & 0xFFFFull) != 0);
            }
        } else if constexpr (FORM == kFormSmall) {
            // Two register buffers in rotation: while the wave hashes and
            // stores one chunk, the next chunk's loads are in flight.  The
            // loop is unrolled by two so that no buffer is ever copied into
            // the other (a copy would wait for its loads).
            uint4 v0[kLoadsInFlight], v1[kLoadsInFlight];
            const Desc *td = desc[buf];
            int t = group;   // uniform over the wave
            SmallItem x, y;
            if (t < cnt) {
                x = small_item<MODE>(td[t]);
                small_loads<MODE, NT>(x, lane, v0);
            }
            while (t < cnt) {
                const int u = groups + take_chunk(&s_next[buf], lane);
                arrived(v0);
                if (u < cnt) {
                    y = small_item<MODE>(td[u]);
                    small_loads<MODE, NT>(y, lane, v1);
                }
                small_chunk<MODE, NT>(a, T, out, t, td[t], x, lane, C, v0);
                if (u >= cnt)
                    break;
                t = groups + take_chunk(&s_next[buf], lane);
                arrived(v1);
                if (t < cnt) {
                    x = small_item<MODE>(td[t]);
                    small_loads<MODE, NT>(x, lane, v0);
                }
                small_chunk<MODE, NT>(a, T, out, u, td[u], y, lane, C, v1);
            }
        } else if constexpr (FORM == kFormLong) {
            // As above, two register buffers in rotation; the load cursor
            // (x, lt, lr) runs one batch ahead of the work cursor (y, t, rb).
            constexpr int B = kLoadsInFlight;
            uint4 v0[B], v1[B];
            const Desc *td = desc[buf];
            int t = group, lt = group;   // uniform over the wave
            if (t < cnt) {
                LongItem x = long_item<MODE>(td[t], r_win, C), y = x;
                uint32_t lr = x.r0, rb = x.r0, acc = 0;
                bool seen = false;
                const auto ahead = [&](uint4 (&v)[B]) {   // loads of the next batch; false after the last
                    lr += B;
                    if (lr >= r_win) {
                        lt = groups + take_chunk(&s_next[buf], lane);
                        if (lt >= cnt)
                            return false;
                        x = long_item<MODE>(td[lt], r_win, C);
                        lr = x.r0;
                    }
                    long_loads<MODE, NT>(x, lane, r_win, lr, v);
                    return true;
                };
                const auto work = [&](uint4 (&v)[B]) {
                    long_batch<MODE, NT>(a, T, out, t, td[t], y, lane, r_win, rb, v, &acc, &seen);
                    rb += B;
                    if (rb >= r_win) {   // x is this wave's next chunk by now, or there is none
                        t = lt;
                        y = x;
                        rb = y.r0;
                        acc = 0;
                        seen = false;
                    }
                };
                long_loads<MODE, NT>(x, lane, r_win, lr, v0);
                for (;;) {
                    arrived(v0);
                    bool more = ahead(v1);
                    work(v0);
                    if (!more)
                        break;
                    arrived(v1);
                    more = ahead(v0);
                    work(v1);
                    if (!more)
                        break;
                }
            }
        } else {
        for (int slot = 0; slot < cnt; slot += groups) {
            const int t = slot + group;
            const bool valid = t < cnt;
            uint32_t raw = 0, orv = 0;
            Desc d;
            if (valid) {
                d = desc[buf][t];
                raw = wave_rounds<MODE, NT>(T, d, lane, wig * rw, (wig + 1) * rw, r_win, &orv);
            }
            const bool nonzero = __ballot(orv != 0) != 0;
            if (lane == 0) {
                s_part[wave] = raw;
                s_nz[wave] = nonzero;
            }
            __syncthreads();
            if (valid && wig == 0) {   // uniform over the wave
                uint32_t acc = s_part[wave];
                bool nz = s_nz[wave];
                for (int w = 1; w < W; w++) {
                    acc = T.seg(acc) ^ s_part[wave + w];
                    nz = nz || s_nz[wave + w];
                }
                const uint32_t crc = finish_crc(T, acc, d.len, lane);
                if (lane == 0)
                    finish_chunk<MODE>(a, out, t, d, crc, nz);
            }
            __syncthreads();
        }
        }
        if (have_nd)
            desc[buf ^ 1][per_tile(threadIdx.x)] = nd;   // the other tile was consumed before the last barrier
        if (threadIdx.x == 0 && nxt < n_tiles) {
            s_tile[(it + 1) & 1] = gridDim.x + taken;   // read after the next barrier
            if (taken >= n_dyn)
                tiles_done(&a.plan_rw->tile_next, taken, n_dyn, gridDim.x);
        }
        if (MODE != kModeRestore && threadIdx.x == 0)
            s_done[row] = cur;
        done = cur;
        cur = nxt;
        its = it + 1;
    }
    __syncthreads();
    put_results(its, done, buf ^ 1, true);
}

template <int MODE, bool NT, int FORM = kFormWave>
__global__ __launch_bounds__(1024) void k_chunks(ChunkArgs a)
{
    chunks<MODE, NT, FORM, false>(a, nullptr);
}

// The same for a table of at most kRowTile rows in its arguments: no kernel
// before it lays the table out (13 buffers of 100 bytes to 256 KiB: 22.3 us a
// call with k_prologue_small before it, 19.1 so).
template <int MODE, bool NT, int FORM = kFormWave>
__global__ __launch_bounds__(1024) void k_chunks_table(ChunkArgs a, SmallTable t)
{
    chunks<MODE, NT, FORM, true>(a, &t);
}

// ------------------------------------------------- row mode (serving loop)
//
// Same per-chunk work as k_chunks (one wave per chunk), but each item's
// addresses come from its row, and each row says whether its chunks are
// packed or restored; the branch is uniform across a wave.

struct RowDesc {
    Desc d;
    uint64_t crc, flags, bad, bad_count;
    uint32_t mode, pad;
};

__device__ __forceinline__ RowDesc make_row_desc(const RowArgs &a, uint64_t i, uint32_t C)
{
    const StepRow &row = a.rows[a.map[i]];
    const uint64_t c = i - row.item0;
    const uint64_t start = c * C;
    const uint64_t rest = row.rem - start;
    RowDesc r;
    r.d.g = i;
    r.d.len = (uint32_t)(rest < C ? rest : C);
    r.d.has_base = 0;
    r.mode = row.mode;
    r.pad = 0;
    r.crc = row.crc + 4 * c;
    r.flags = row.flags + c;
    r.bad = row.bad + c;
    r.bad_count = row.bad_count;
    if (row.mode == kModeRestore) {
        r.d.zero = *(Global<const uint8_t> *)r.flags & kFlagZero;
        r.d.want = *(Global<const uint32_t> *)r.crc;
        r.d.src = r.d.zero ? 0 : row.src + ((Global<const uint64_t> *)row.soff)[c];
    } else {
        r.d.zero = 0;
        r.d.want = 0;
        r.d.src = row.src + start;
    }
    r.d.dst = row.dst + start;
    return r;
}

template <bool NT>
__global__ __launch_bounds__(1024) void k_rows(RowArgs a)
{
    __shared__ __attribute__((aligned(16))) uint32_t tabs[kRepWords];
    __shared__ RowDesc desc[2][kRowsTile];

    stage_tables(tabs, a.tables, [] {});
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const Tabs T = make_tabs(tabs, lane);
    const int nwaves = blockDim.x >> 6;
    const uint32_t C = a.C;
    const uint32_t r_win = (C + kRoundBytes - 1) / kRoundBytes;
    const uint64_t M = a.n_items;

    // Tiles taken from the step's counter, one ahead, and double-buffered
    // descriptors, as in k_chunks.
    const uint64_t n_tiles = (M + kRowsTile - 1) / kRowsTile;
    const bool stager = threadIdx.x < kRowsTile;
    __shared__ uint64_t s_tile[2];
    if (threadIdx.x == 0) {
        const uint64_t c = take_tile(a.tile_ctr);
        uint64_t n = n_tiles;
        if (c < n_tiles)
            n = take_tile(a.tile_ctr);
        if (c >= n_tiles)
            tiles_done(a.tile_ctr, c, n_tiles, gridDim.x);
        else if (n >= n_tiles)
            tiles_done(a.tile_ctr, n, n_tiles, gridDim.x);
        s_tile[0] = c;
        s_tile[1] = n;
    }
    __syncthreads();
    uint64_t cur = s_tile[0], nxt = s_tile[1];
    if (cur < n_tiles && stager && cur * kRowsTile + threadIdx.x < M)
        desc[0][threadIdx.x] = make_row_desc(a, cur * kRowsTile + threadIdx.x, C);
    int buf = 0;
    for (uint32_t it = 0; cur < n_tiles; it++, buf ^= 1) {
        __syncthreads();
        if (it > 0)
            nxt = s_tile[(it + 1) & 1];
        uint64_t taken = n_tiles;
        if (threadIdx.x == 0 && nxt < n_tiles)
            taken = take_tile(a.tile_ctr);
        const uint64_t g0 = cur * kRowsTile, hi = g0 + kRowsTile < M ? g0 + kRowsTile : M;
        const uint64_t n0 = nxt * kRowsTile, n1 = nxt < n_tiles ? (n0 + kRowsTile < M ? n0 + kRowsTile : M) : n0;
        RowDesc nd;
        if (stager && n0 + threadIdx.x < n1)
            nd = make_row_desc(a, n0 + threadIdx.x, C);
        const int cnt = (int)(hi - g0);
        for (int t = wave; t < cnt; t += nwaves) {
            const RowDesc rd = desc[buf][t];
            uint32_t raw, orv;
            if (rd.mode == kModeRestore)
                raw = wave_rounds<kModeRestore, NT>(T, rd.d, lane, 0, r_win, r_win, &orv);
            else
                raw = wave_rounds<kModePack, NT>(T, rd.d, lane, 0, r_win, r_win, &orv);
            const bool nonzero = __ballot(orv != 0) != 0;
            const uint32_t crc = finish_crc(T, uniform_u32(raw), rd.d.len, lane);
            if (lane == 0) {
                if (rd.mode == kModeRestore) {
                    if (crc != rd.d.want) {
                        *(Global<uint8_t> *)rd.bad = 1;
                        atomicAdd((unsigned long long *)rd.bad_count, 1ull);
                    }
                } else {
                    *(Global<uint32_t> *)rd.crc = crc;
                    *(Global<uint8_t> *)rd.flags = (nonzero ? 0 : kFlagZero) | kFlagDirty;
                }
            }
        }
        if (stager && n0 + threadIdx.x < n1)
            desc[buf ^ 1][threadIdx.x] = nd;
        if (threadIdx.x == 0 && nxt < n_tiles) {
            s_tile[it & 1] = taken;
            if (taken >= n_tiles)
                tiles_done(a.tile_ctr, taken, n_tiles, gridDim.x);
        }
        cur = nxt;
    }
}

// ------------------------------------------------------ K5: selection scan
//
// Reduce-then-scan over items in tiles of kSelTile.  Per item: `bytes`
// (roundup16 of the chunk's length when the chunk is selected) and `count` (1
// when its id goes to the id list).  soff[i] gets the exclusive prefix of
// bytes; ids_out gets the counted ids in ascending order.
//   Totals per tile: a pack or hash pass adds up its chunks' itself
//   (k_chunks); else k_sel_reduce.  A tile's share is bytes in the low 48 bits
//   (at most 4096 chunks of 2^30 bytes) and count above.
//   k_sel_down: each workgroup adds up the totals before its tile and scans the
//   tile.  Beyond kSelDirect tiles, where that would be more than the scan's
//   own traffic, k_sel_scan makes the prefix sums first.
// Bound by latency: as three launches with the totals copied to the host by a
// fourth it took 27 us between a drain's pack and its gather.

__device__ __forceinline__ uint64_t sel_items(const SelArgs &a)
{
    return a.n_known ? a.n_known : a.plan->n_chunks;
}

// roundup16 of chunk g's length; g is not the last of its row when its
// successor has the same row.
__device__ __forceinline__ uint64_t sel_len(const SelArgs &a, uint64_t g, uint32_t k, bool last)
{
    if (!last)
        return a.C;
    const uint64_t rest = a.size[k] - (g - a.cb[k]) * a.C;
    return round_up16(rest < a.C ? rest : a.C);
}

// The thread's kSelPerThread items from i0 on: b[j] and the bits of `id`;
// ids in g[j] (mode kSelIdsNonZero).
__device__ __forceinline__ void sel_load(const SelArgs &a, uint64_t i0, uint64_t M, uint64_t (&b)[kSelPerThread],
                                         uint32_t *id)
{
    static_assert(kSelPerThread == 16, "16 flags are one load");
    *id = 0;
    if (a.mode == kSelIdsNonZero || i0 + kSelPerThread >= M) {   // ids, or the end of the items
        for (int j = 0; j < kSelPerThread; j++) {
            const uint64_t i = i0 + j;
            b[j] = 0;
            if (i >= M)
                continue;
            const uint64_t g = a.mode == kSelIdsNonZero ? a.ids[i] : i;
            bool take, c;
            sel_flags(a.mode, a.flags[g], &take, &c);
            if (take)
                b[j] = sel_len(a, g, a.map[g], true);
            *id |= (uint32_t)c << j;
        }
        return;
    }
    const uint4 fq = *(const uint4 *)(a.flags + i0);
    const uint32_t f[4] = {fq.x, fq.y, fq.z, fq.w};
    uint32_t k[kSelPerThread + 1];
#pragma unroll
    for (int j = 0; j < kSelPerThread; j += 4) {
        const uint4 q = *(const uint4 *)(a.map + i0 + j);
        k[j] = q.x;
        k[j + 1] = q.y;
        k[j + 2] = q.z;
        k[j + 3] = q.w;
    }
    k[kSelPerThread] = a.map[i0 + kSelPerThread];
#pragma unroll
    for (int j = 0; j < kSelPerThread; j++) {
        bool take, c;
        sel_flags(a.mode, (uint8_t)(f[j / 4] >> (8 * (j % 4))), &take, &c);
        b[j] = take ? sel_len(a, i0 + j, k[j], k[j] != k[j + 1]) : 0;
        *id |= (uint32_t)c << j;
    }
}

// Block-wide exclusive scan of (bytes, count) pairs; returns the block totals.
__device__ __forceinline__ void block_excl_scan(uint64_t &b, uint64_t &c, uint64_t *tot_b, uint64_t *tot_c)
{
    __shared__ uint64_t sb[16], sc[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint64_t ib = wave_incl_scan(b, lane), ic = wave_incl_scan(c, lane);
    if (lane == 63) {
        sb[wave] = ib;
        sc[wave] = ic;
    }
    __syncthreads();
    uint64_t pb = 0, pc = 0, tb = 0, tc = 0;
    for (int w = 0; w < nw; w++) {
        if (w < wave) {
            pb += sb[w];
            pc += sc[w];
        }
        tb += sb[w];
        tc += sc[w];
    }
    __syncthreads();
    b = pb + ib - b;
    c = pc + ic - c;
    *tot_b = tb;
    *tot_c = tc;
}

__global__ __launch_bounds__(kSelThreads) void k_sel_reduce(SelArgs a)
{
    const uint64_t M = sel_items(a);
    const uint64_t first = (uint64_t)blockIdx.x * kSelTile;
    uint64_t b = 0, c = 0;
    if (first < M) {
        uint64_t ib[kSelPerThread];
        uint32_t id;
        sel_load(a, first + (uint64_t)threadIdx.x * kSelPerThread, M, ib, &id);
        for (int j = 0; j < kSelPerThread; j++)
            b += ib[j];
        c = __popc(id);
    }
    uint64_t tb, tc;
    block_excl_scan(b, c, &tb, &tc);
    if (threadIdx.x == 0)
        a.tile_bytes[blockIdx.x] = sel_pack(tb, tc);
}

__global__ __launch_bounds__(1024) void k_sel_scan(SelArgs a)
{
    const uint64_t M = sel_items(a);
    const uint64_t tiles = (M + kSelTile - 1) / kSelTile;
    uint64_t carry_b = 0, carry_c = 0;
    for (uint64_t base = 0; base < tiles; base += 1024) {
        const uint64_t t = base + threadIdx.x;
        const uint64_t v = t < tiles ? a.tile_bytes[t] : 0;
        uint64_t b = sel_bytes(v), c = sel_count(v);
        uint64_t tb, tc;
        block_excl_scan(b, c, &tb, &tc);
        if (t < tiles) {
            a.tile_bytes[t] = carry_b + b;
            a.tile_count[t] = carry_c + c;
        }
        carry_b += tb;
        carry_c += tc;
    }
}

__global__ __launch_bounds__(kSelThreads) void k_sel_down(SelArgs a)
{
    const uint64_t M = sel_items(a);
    const uint64_t tiles = (M + kSelTile - 1) / kSelTile;
    if (blockIdx.x >= tiles && blockIdx.x > 0)
        return;
    // the totals of the tiles before this one
    uint64_t base_b = 0, base_c = 0;
    if (a.scanned) {
        if (tiles) {
            base_b = a.tile_bytes[blockIdx.x];
            base_c = a.tile_count[blockIdx.x];
        }
    } else {
        uint64_t b = 0, c = 0;
        for (uint64_t t = threadIdx.x; t < blockIdx.x; t += kSelThreads) {
            const uint64_t v = a.tile_bytes[t];
            b += sel_bytes(v);
            c += sel_count(v);
        }
        block_excl_scan(b, c, &base_b, &base_c);
    }
    const uint64_t i0 = (uint64_t)blockIdx.x * kSelTile + (uint64_t)threadIdx.x * kSelPerThread;
    uint64_t ib[kSelPerThread];
    uint32_t id;
    sel_load(a, i0, M, ib, &id);
    uint64_t b = 0, c = __popc(id);
#pragma unroll
    for (int j = 0; j < kSelPerThread; j++)
        b += ib[j];
    uint64_t tb, tc;
    block_excl_scan(b, c, &tb, &tc);
    if (blockIdx.x + 1 >= tiles && threadIdx.x == 0) {   // the last tile (or the only workgroup)
        a.plan->sel_bytes = base_b + tb;
        a.plan->sel_count = base_c + tc;
        if (a.want_id && a.want != base_b + tb && !a.plan->sel_bad) {
            a.plan->sel_bad = a.want_id;
            a.plan->sel_found = base_b + tb;
        }
        if (a.h_plan) {
            a.h_plan->sel_bytes = base_b + tb;
            a.h_plan->sel_count = base_c + tc;
        }
    }
    b += base_b;
    c += base_c;
    if (a.soff) {
        uint64_t o = b;
        if (i0 + kSelPerThread <= M) {
#pragma unroll
            for (int j = 0; j < kSelPerThread; j += 2) {
                *(ulonglong2 *)(a.soff + i0 + j) = make_ulonglong2(o, o + ib[j]);
                o += ib[j] + ib[j + 1];
            }
        } else {
            for (int j = 0; j < kSelPerThread && i0 + j < M; j++) {
                a.soff[i0 + j] = o;
                o += ib[j];
            }
        }
    }
    if (a.ids_out)
        for (; id; id &= id - 1) {
            const uint64_t i = i0 + __builtin_ctz(id);
            if (c < a.ids_cap)
                a.ids_out[c] = a.mode == kSelIdsNonZero ? a.ids[i] : i;
            c++;
        }
}

// --------------------------------------------------------------- K6: gather
//
// Copies each selected chunk (roundup16(len) bytes) to out + soff[g], from the
// dense image or straight from the allocation (zero pad written, never read);
// or, for several outputs in host memory, into each output's own buffer.
// Bound by HBM (by the host link when the output is host memory).  A workgroup
// takes tiles of consecutive chunks, one per thread for the descriptors; the
// selected ones are compacted into a list in LDS, and its waves then copy the
// list's pieces of at most 4 KiB in turn, each lane with up to
// kGatherLoads 16-byte loads before its first store.  So a tile with few
// selected chunks, or with large ones, still occupies every wave.
// The tile follows from the launch: about two per workgroup, 16 to 1024
// chunks.  Small launches then use the whole grid: with fixed tiles of 1024
// chunks (64 per wave, each wave copying its own chunks whole), 9 MB in 2350
// chunks ran on 3 workgroups.  The list's pieces are counted by the chunks' own
// lengths: with as many units for each as a full chunk has, an increment of 300
// allocations of 1000 bytes took 10.4 ms with chunks of 256 MiB, now 82 us.

constexpr int kGatherLoads = 4;
constexpr uint32_t kGatherPiece = kGatherLoads * 1024;
constexpr int kGatherTile = 1024;   // most chunks per tile: one per thread
constexpr int kGatherMinTile = 16;

// n <= kGatherPiece bytes, by one wave.
template <bool NT_ST>
__device__ __forceinline__ void gather_copy(const uint8_t *s, uint8_t *d, uint32_t n, bool whole, int lane)
{
    uint4 v[kGatherLoads];
#pragma unroll
    for (int u = 0; u < kGatherLoads; u++) {
        const uint32_t o = 16 * (uint32_t)(u * 64 + lane);
        v[u] = make_uint4(0u, 0u, 0u, 0u);
        if (o < n) {   // past an allocation's tail the piece's bytes are not the chunk's (see load_piece)
            v[u] = ld16<true>(s + o);
            if (!whole && o + 16 > n)
                v[u] = keep_bytes(v[u], n - o);
        }
    }
#pragma unroll
    for (int u = 0; u < kGatherLoads; u++) {
        const uint32_t o = 16 * (uint32_t)(u * 64 + lane);
        if (o < n)
            st16<NT_ST>(d + o, v[u]);
    }
}

// The chunk of a list that unit u belongs to: the last of the `cnt` (at most
// kGatherTile) whose first unit is at most u.  By the whole wave: every 16th
// chunk, then the 16 from there on.
__device__ __forceinline__ uint32_t gather_chunk(const uint32_t *first, uint32_t cnt, uint32_t u, int lane)
{
    static_assert(kGatherTile <= 64 * 16, "two steps");
    const uint32_t i = 16 * (uint32_t)lane;
    const uint32_t b = 16 * (uint32_t)(__popcll(__ballot(i < cnt && first[i] <= u)) - 1);
    const uint32_t j = b + (uint32_t)lane;
    return b + (uint32_t)__popcll(__ballot(lane < 16 && j < cnt && first[j] <= u)) - 1;
}

template <bool NT_ST>
__global__ __launch_bounds__(1024) void k_gather(GatherArgs a)
{
    __shared__ uint64_t s_t[2];
    __shared__ uint64_t s_src[kGatherTile], s_dst[kGatherTile];
    __shared__ uint32_t s_len[kGatherTile];
    __shared__ uint32_t s_first[kGatherTile];   // units (pieces) before the chunk's
    __shared__ uint32_t s_cnt[16], s_units[16];
    const uint64_t N = a.g_end ? a.g_end : a.plan->n_chunks;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint64_t total = N > a.g_begin ? N - a.g_begin : 0;
    uint32_t span = kGatherTile;   // chunks per tile
    while (span > kGatherMinTile && (uint64_t)span * 2 * gridDim.x > total)
        span >>= 1;
    const uint64_t n_tiles = (total + span - 1) / span;
    const bool one_piece = a.C <= kGatherPiece;   // then unit u is the list's chunk u
    // Workgroup b's first tile is tile b; the rest are taken in order from the
    // plan's counter by thread 0, so that a workgroup whose tiles hold few
    // selected chunks takes more of them.
    const uint64_t n_dyn = n_tiles > gridDim.x ? n_tiles - gridDim.x : 0;
    for (uint32_t c = 0; c < a.n_copy; c++)
        copy_span(a.copy[c], (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, (uint64_t)gridDim.x * blockDim.x);
    for (uint32_t it = 0;; it++) {
        if (threadIdx.x == 0) {
            uint64_t t = n_tiles;
            if (it == 0) {
                t = blockIdx.x;
            } else if (n_dyn) {
                const uint64_t v = take_tile(a.tile_ctr);
                if (v >= n_dyn)
                    tiles_done(a.tile_ctr, v, n_dyn, gridDim.x);
                t = gridDim.x + v;
            }
            s_t[it & 1] = t;   // the other slot may still be read
        }
        __syncthreads();   // every wave has copied its part of the previous list
        const uint64_t cur = s_t[it & 1];
        if (cur >= n_tiles)
            break;
        const uint64_t g = a.g_begin + cur * span + threadIdx.x;
        bool take = false;
        uint64_t src = 0, dst = 0;
        uint32_t len = 0;
        if (threadIdx.x < span && g < N) {
            const uint8_t f = a.flags[g];
            const uint32_t k = a.map[g];
            const uint64_t so = a.soff[g];
            take = a.mode == kSelNonZero ? !(f & kFlagZero) : ((f & kFlagDirty) && !(f & kFlagZero));
            if (take) {
                const uint64_t start = (g - a.cb[k]) * a.C;
                const uint64_t rest = a.size[k] - start;
                len = (uint32_t)(rest < a.C ? rest : a.C);
                src = a.from_dense ? (uint64_t)(a.dense + a.off[k] + start) : a.src[k] + start;
                if (a.out_addr) {
                    const uint32_t o = a.row_out[k];
                    dst = a.out_addr[o] + (so - a.soff[a.out_chunk0[o]]);
                } else {
                    dst = (uint64_t)(a.out + (so - a.soff_base));
                }
            }
        }
        const uint64_t m = __ballot(take);
        // units by the chunks' own lengths: a tile of short chunks has few, whatever C is
        const uint32_t mine = one_piece ? 0 : (len + kGatherPiece - 1) / kGatherPiece;
        uint32_t upto = mine;
        if (!one_piece) {
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t v = __shfl_up(upto, d, 64);
                upto += lane >= d ? v : 0;
            }
        }
        if (lane == 63) {
            s_cnt[wave] = (uint32_t)__popcll(m);
            s_units[wave] = upto;
        }
        __syncthreads();
        uint32_t pos = 0, cnt = 0, first = upto - mine, units = 0;
        for (int w = 0; w < nw; w++) {
            if (w == wave) {
                pos = cnt;
                first += units;
            }
            cnt += s_cnt[w];
            units += s_units[w];
        }
        if (one_piece)
            units = cnt;
        if (take) {
            pos += (uint32_t)__popcll(m & ((1ull << lane) - 1));
            s_src[pos] = src;
            s_dst[pos] = dst;
            s_len[pos] = len;
            s_first[pos] = first;
        }
        __syncthreads();
        for (uint32_t u = wave; u < units; u += nw) {   // uniform over the wave
            const uint32_t c = one_piece ? u : gather_chunk(s_first, cnt, u, lane);
            const uint32_t o = one_piece ? 0 : (u - uniform_u32(s_first[c])) * kGatherPiece;
            const uint32_t n = uniform_u32(s_len[c]) - o;
            gather_copy<NT_ST>((const uint8_t *)uniform_u64(s_src[c]) + o, (uint8_t *)uniform_u64(s_dst[c]) + o,
                               n < kGatherPiece ? n : kGatherPiece, a.from_dense != 0, lane);
        }
    }
}

// ------------------------------------------------------------------ helpers

// The allocation table as the host keeps it (rows of four words: id, kind,
// address, size) split into the address and size arrays the scan and the
// chunk kernels read; the first thread also writes a fresh plan for n rows.
__global__ void k_table_split(const uint64_t *__restrict__ rows, uint64_t n, DevPlan *plan,
                              uint64_t *__restrict__ addr, uint64_t *__restrict__ size)
{
    const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i0 == 0) {
        DevPlan p = {};
        p.n_allocs = n;
        *plan = p;
    }
    for (uint64_t k = i0; k < n; k += (uint64_t)gridDim.x * blockDim.x) {
        addr[k] = rows[4 * k + 2];
        size[k] = rows[4 * k + 3];
    }
}

__global__ void k_pick_u64(const uint64_t *src, const uint64_t *idx, uint64_t *out, uint32_t m)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m)
        out[i] = src[idx[i]];
}

// ----------------------------------------------------------- launch wrappers

hipError_t launch_prologue(hipStream_t s, const PrologueArgs &a, uint64_t items)
{
    const uint64_t grid = items < 1 ? 1 : items > 2048 ? 2048 : items;
    hipLaunchKernelGGL(k_prologue, dim3((unsigned)grid), dim3(kPrologueThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_prologue_small(hipStream_t s, const PrologueArgs &a, const SmallTable &t)
{
    hipLaunchKernelGGL(k_prologue_small, dim3(1), dim3(1024), 0, s, a, t);
    return hipGetLastError();
}

hipError_t launch_layout_scan(hipStream_t s, DevPlan *plan, const uint64_t *size, uint32_t C, uint64_t *off,
                              uint64_t *cb)
{
    hipLaunchKernelGGL(k_layout_scan, dim3(1), dim3(1024), 0, s, plan, size, C, off, cb);
    return hipGetLastError();
}

hipError_t launch_chunk_map(hipStream_t s, const DevPlan *plan, const uint64_t *cb, uint32_t *map, int grid)
{
    hipLaunchKernelGGL(k_chunk_map, dim3(grid), dim3(256), 0, s, plan, cb, map);
    return hipGetLastError();
}

template <int MODE, int FORM>
static void launch_form(hipStream_t s, const ChunkArgs &a, const SmallTable *t, int grid, int block)
{
    if constexpr (MODE != kModeRestore) {
        if (t) {
            if (a.nontemporal)
                hipLaunchKernelGGL((k_chunks_table<MODE, true, FORM>), dim3(grid), dim3(block), 0, s, a, *t);
            else
                hipLaunchKernelGGL((k_chunks_table<MODE, false, FORM>), dim3(grid), dim3(block), 0, s, a, *t);
            return;
        }
    }
    if (a.nontemporal)
        hipLaunchKernelGGL((k_chunks<MODE, true, FORM>), dim3(grid), dim3(block), 0, s, a);
    else
        hipLaunchKernelGGL((k_chunks<MODE, false, FORM>), dim3(grid), dim3(block), 0, s, a);
}

template <int MODE>
static void launch_chunks_m(hipStream_t s, const ChunkArgs &a, const SmallTable *t, int grid, int block)
{
    const uint32_t rounds = (a.C + kRoundBytes - 1) / kRoundBytes;
    // hash-only chunks of at most 4 KiB: four chunks per wave
    if constexpr (MODE == kModeHash) {
        if (a.tables_quad && a.waves_per_chunk == 1 && rounds <= kQuadMaxRounds) {
            ChunkArgs q = a;
            q.tables = a.tables_quad;
            launch_form<kModeHash, kFormQuad>(s, q, t, grid, block);
            return;
        }
    }
    // one wave per chunk: one batch of rounds per chunk, or several
    if (a.waves_per_chunk == 1 && rounds <= kLoadsInFlight)
        launch_form<MODE, kFormSmall>(s, a, t, grid, block);
    else if (a.waves_per_chunk == 1)
        launch_form<MODE, kFormLong>(s, a, t, grid, block);
    else
        launch_form<MODE, kFormWave>(s, a, t, grid, block);
}

hipError_t launch_chunks(hipStream_t s, int mode, const ChunkArgs &a, int grid, int block)
{
    switch (mode) {
    case kModePack: launch_chunks_m<kModePack>(s, a, nullptr, grid, block); break;
    case kModeHash: launch_chunks_m<kModeHash>(s, a, nullptr, grid, block); break;
    default: launch_chunks_m<kModeRestore>(s, a, nullptr, grid, block); break;
    }
    return hipGetLastError();
}

bool table_fits(uint64_t n_rows, uint64_t n_chunks, int grid)
{
    return n_rows && n_rows <= kRowTile && n_chunks <= (uint64_t)grid * kTile;
}

hipError_t launch_chunks_table(hipStream_t s, int mode, const ChunkArgs &a, const SmallTable &t, int grid, int block)
{
    if (mode == kModePack)
        launch_chunks_m<kModePack>(s, a, &t, grid, block);
    else
        launch_chunks_m<kModeHash>(s, a, &t, grid, block);
    return hipGetLastError();
}

hipError_t launch_rows(hipStream_t s, const RowArgs &a, int grid, int block)
{
    if (a.nontemporal)
        hipLaunchKernelGGL((k_rows<true>), dim3(grid), dim3(block), 0, s, a);
    else
        hipLaunchKernelGGL((k_rows<false>), dim3(grid), dim3(block), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_select(hipStream_t s, const SelArgs &a_in, uint64_t max_items, bool have_totals)
{
    SelArgs a = a_in;
    const uint64_t tiles = (max_items + kSelTile - 1) / kSelTile;
    const unsigned grid = (unsigned)(tiles ? tiles : 1);
    // one tile has no totals before it to add (a refill of 2300 chunks: 221 us
    // with the launch, 214 without)
    if (!have_totals && tiles > 1)
        hipLaunchKernelGGL(k_sel_reduce, dim3(grid), dim3(kSelThreads), 0, s, a);
    a.scanned = tiles > kSelDirect;
    if (a.scanned)
        hipLaunchKernelGGL(k_sel_scan, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(k_sel_down, dim3(grid), dim3(kSelThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_gather(hipStream_t s, const GatherArgs &a_in, int grid)
{
    GatherArgs a = a_in;
    a.tile_ctr = (unsigned long long *)((uintptr_t)a.plan + offsetof(DevPlan, gather_next));
    // stores into pinned host memory (the direct drain) keep the default policy
    if (a.out_host)
        hipLaunchKernelGGL(k_gather<false>, dim3(grid), dim3(1024), 0, s, a);
    else
        hipLaunchKernelGGL(k_gather<true>, dim3(grid), dim3(1024), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_table_split(hipStream_t s, const uint64_t *rows, uint64_t n, DevPlan *plan, uint64_t *addr,
                              uint64_t *size)
{
    uint64_t blocks = (n + 255) / 256;
    blocks = blocks < 1 ? 1 : blocks > 1024 ? 1024 : blocks;
    hipLaunchKernelGGL(k_table_split, dim3((unsigned)blocks), dim3(256), 0, s, rows, n, plan, addr, size);
    return hipGetLastError();
}

hipError_t launch_pick_u64(hipStream_t s, const uint64_t *src, const uint64_t *idx, uint64_t *out, uint32_t m)
{
    if (m == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_pick_u64, dim3((m + 255) / 256), dim3(256), 0, s, src, idx, out, m);
    return hipGetLastError();
}

}  // namespace ckpt

// The level sweep for circuits with few gates per level, with the HEADS of a tile spread over compute units.
//
// On such circuits (a few hundred gates per dependency level, any number of levels) the sweep is bound by
// the time from a gate to its reader, and a kernel that gives a whole tile to one compute unit spends that
// time streaming weights (512 bytes x 4 x hidden per layer through one unit's vector memory path) and
// gathering whole K | V rows, while most units idle. Here a tile of at most 16 gates is worked on by
// C = hidden / 32 workgroups, one per head ("slice"); workgroup b takes slice b % C, and since workgroups
// are dealt to the eight XCDs in turn, an XCD sees one slice only (hidden 256) or shares one with a second
// XCD (hidden 128). Per layer a slice
//   - attends with its head: its part of the state's Q | K | V (96 columns, projected here), its part of
//     the sources' K | V rows. The store of finished gates is kept per slice, K | V of a head side by
//     side in 128 (bf16) or 256 (fp32) bytes, so an XCD's L2 holds 1/C of every row instead of all of
//     some, and the gates of a level that read the same source share it there;
//   - hands its 32 columns of the attention output to the other slices and collects theirs: 64-bit words of
//     32 bits of data and a 32-bit tag, written and polled with agent-scope accesses, so that one trip
//     through memory carries data and "ready" together (a word is written whole or not at all);
//   - forms the output projection, residual and LayerNorm of whole rows (every slice the same bits), from
//     which its part of the next layer's Q | K | V follows without another exchange.
// Behind the last layer a slice projects its head's K | V of every layer and raises its own flag; readers
// of a slice wait for flags of that slice only. With the feed-forward sub-block a slice forms 128 of the
// 4d activations, collects the rest, forms 32 output columns (the products over 4d split over the eight
// waves) and collects the others' before the second LayerNorm.
//
// Weights per layer and workgroup: Wo whole and 96 columns of Wq | Wk | Wv, every wave's fragments requested
// one phase ahead into registers, so that a product waits for no memory.
//
// Order and progress: C workgroups, one per slice, form a GROUP and run through the same tiles together; its
// slice 0 draws the tickets (one counter over the list of tiles) and hands them to the others through a mailbox word.
// Groups consist of workgroups that run (dg4_sit), so a ticket is only ever held by workgroups that run, and a tile
// waits for lower tickets only: the lowest unfinished tile always advances as long as one group has formed. First C
// workgroups with consecutive numbers look for each other (an XCD then sees one slice); should one of them not turn
// up, because other work holds its compute units, the rest close the group and sit down in the order they come in,
// each taking the slice of its place, so any C workgroups that run make a group, whatever else the device is
// doing. Groups that never fill leave when the tickets have run out. A bounded spin count turns
// any violation into an abort word. The exchange words of a group alternate between two places: a slice
// writes the words of round k + 2 only after it has collected round k + 1 from all the others, each of which
// had read round k before. (Tickets per slice, without groups, measured 11 us more per tile: the slices of a
// tile then start whenever their workgroups happen to be free.)
//
// Visibility: K | V rows are written once per sweep with agent-scope stores that have completed before the
// flag goes up, flags and exchange words are read with agent-scope loads, and no row is read before its
// flag has been seen (as in the other persistent kernels).
#include <hip/hip_runtime.h>
#include <float.h>
#include <stdint.h>

#include "dg4_device.h"
#include "dg4_internal.h"
#include "dg4_rowops.h"
#include "dg4_wait.h"

namespace {

constexpr int HT = 512;                       // threads (eight waves)
constexpr int HR = DG4_HEADS_ROWS;            // most gates of a tile (one block of 16 of the matrix cores)
// words (32 bits) of the sync area: ticket counters of the finished gates' tiles per slice, the ticket counter of
// the sweep, the number of groups formed and of workgroups that look for another group, the words of the groups by
// workgroup number and by order of arrival, and the (64-bit) mailboxes, every one 64 bytes from the next
static_assert(256 / 4 <= DG4_HEADS_GROUPS, "groups of the smaller number of heads");
constexpr int SYNC_TICKET = 8 * 16, SYNC_FORMED = 9 * 16, SYNC_LOOSE = 10 * 16, SYNC_GROUP = 11 * 16,
              SYNC_REGROUP = SYNC_GROUP + DG4_HEADS_GROUPS * 16, SYNC_MAIL = SYNC_REGROUP + DG4_HEADS_GROUPS * 16;
static_assert((SYNC_MAIL + DG4_HEADS_GROUPS * 16) * 4 <= DG4_HEADS_SYNC_BYTES, "sync area");

template <typename T> struct HeadMma;
template <> struct HeadMma<bf16_t> {
    __device__ static __forceinline__ void run(const uint4& w, const uint4& r, f32x4& c)
    {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, r), c, 0, 0, 0);
    }
};
template <> struct HeadMma<float> {
    __device__ static __forceinline__ void run(const uint4& w, const uint4& r, f32x4& c)
    {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.x), __uint_as_float(r.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.y), __uint_as_float(r.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.z), __uint_as_float(r.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.w), __uint_as_float(r.w), c, 0, 0, 0);
    }
};

template <int N> __device__ __forceinline__ float ror(float x)        // rotated by N inside each row of 16 lanes
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + N, 0xF, 0xF, true));
}
// the other quad of each eight lanes
__device__ __forceinline__ float xor4(float x)
{
    const int mirrored = __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xF, 0xF, true);    // lane i of eight: 7 - i
    return __int_as_float(__builtin_amdgcn_update_dpp(0, mirrored, 0x1B, 0xF, 0xF, true));            // a quad's lanes turned round
}
// lane J of each quad
template <int J> __device__ __forceinline__ float of_quad(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), J * 0x55, 0xF, 0xF, true));
}
// d[0..3] summed over the lanes of each quad: lane j of the quad ends with the sum of d[j]
__device__ __forceinline__ float quad_sums(const float* d, bool odd, bool upper)
{
    const float a = (odd ? d[1] : d[0]) + xor1(odd ? d[0] : d[1]);
    const float b = (odd ? d[3] : d[2]) + xor1(odd ? d[2] : d[3]);
    return (upper ? b : a) + xor2(upper ? a : b);
}

// A lane's 16 bytes of a row: 8 bfloat16 or 4 floats
template <typename T> struct Bits16;
template <> struct Bits16<float> {
    __device__ static __forceinline__ void unpack(const uint4& v, float* f)
    {
        f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
    }
    __device__ static __forceinline__ uint4 pack(const float* f)
    {
        return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
    }
    __device__ static __forceinline__ float dot(const uint4& a, const uint4& b)
    {
        float d = __uint_as_float(a.x) * __uint_as_float(b.x);
        d = fmaf(__uint_as_float(a.y), __uint_as_float(b.y), d);
        d = fmaf(__uint_as_float(a.z), __uint_as_float(b.z), d);
        return fmaf(__uint_as_float(a.w), __uint_as_float(b.w), d);
    }
    // eight lanes hold a head: side by side, or (APART) the quads q and q + 2 of a row of 16 lanes
    template <bool APART> __device__ static __forceinline__ float head_sum(float p)
    {
        p += xor1(p); p += xor2(p);
        return APART ? quads_sum(p) : p + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(p), 0x141, 0xF, 0xF, true));
    }
    __device__ static __forceinline__ float quads_sum(float p) { return p + ror<8>(p); }
};
template <> struct Bits16<bf16_t> {
    __device__ static __forceinline__ void unpack(const uint4& v, float* f)
    {
        const uint32_t w[4] = { v.x, v.y, v.z, v.w };
#pragma unroll
        for (int i = 0; i < 4; ++i) { f[2 * i] = bf16_lo(w[i]); f[2 * i + 1] = bf16_hi(w[i]); }
    }
    __device__ static __forceinline__ uint4 pack(const float* f)
    {
        return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
    }
    __device__ static __forceinline__ float dot(const uint4& a, const uint4& b)
    {
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
        auto d2 = [](uint32_t x, uint32_t y, float c) {
            return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, x), __builtin_bit_cast(bf16x2_t, y), c, false);
        };
        float d0 = d2(a.x, b.x, 0.f), d1 = d2(a.y, b.y, 0.f);
        d0 = d2(a.z, b.z, d0); d1 = d2(a.w, b.w, d1);
        return d0 + d1;
    }
    template <bool> __device__ static __forceinline__ float head_sum(float p) { p += xor1(p); p += xor2(p); return p; }    // a quad holds a head
    __device__ static __forceinline__ float quads_sum(float p) { return p; }
};

// lanes 16 apart / 32 apart added or compared, the result in both
__device__ __forceinline__ float add16(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}
__device__ __forceinline__ float add32(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}
__device__ __forceinline__ float max16(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float max32(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}

// 16 bytes written through to device memory (agent scope); not tracked by the compiler's wait counting: the
// kernel waits with vmcnt(0) before it raises flags. (The idle cycles keep the next vector instruction from
// overwriting the data registers while the store still reads them.)
typedef uint32_t heads_u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void heads_store16(void* dst, const uint4& v)
{
    const heads_u32x4 t = { v.x, v.y, v.z, v.w };
    __asm__ volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(dst), "v"(t) : "memory");
}

// A value the compiler cannot see through: what is derived from it is computed where it is used and not kept in
// registers across the loops (there are more such values than registers)
__device__ __forceinline__ int fresh(int x)
{
    __asm__ volatile("" : "+v"(x));
    return x;
}
// LDS traffic only: what travels from memory (weights requested ahead) stays in flight
__device__ __forceinline__ void heads_barrier()
{
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);           // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");
}

__device__ __forceinline__ void put_word(uint64_t* dst, uint32_t data, uint32_t tag)
{
    __hip_atomic_store(dst, (uint64_t)tag << 32 | data, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T, int D, int W> struct HeadsLds {            // byte offsets in dynamic LDS
    static constexpr int E = 16 / (int)sizeof(T);
    static constexpr int YS = D + E, QS = 96 + E, US = 4 * D + E;
    static constexpr size_t ROWS = (size_t)HR * YS * sizeof(T);
    static constexpr size_t QKV = (size_t)HR * QS * sizeof(T);
    static constexpr size_t STAT = 2 * (size_t)16 * HR * sizeof(float);
    static constexpr size_t ATT = (size_t)HR * (32 + 2) * sizeof(float);
    static constexpr size_t CTL = 64 + DG4_MAX_LAYERS * 4 * sizeof(float);
    static constexpr size_t off_qkv = 2 * ROWS, off_stat = off_qkv + QKV, off_att = off_stat + STAT, off_ctl = off_att + ATT,
                            off_ticks = off_ctl + CTL, off_ent = off_ticks + 80;
    // words of a neighbour row (W == 0): whole rounds, in which every lane group of the gate takes eight entries
    __host__ __device__ static constexpr int round_words(int tile_rows) { return 8 * (HT / tile_rows) / (32 * (int)sizeof(T) / 16); }
    __host__ __device__ static constexpr int row_words(int ell_w, int tile_rows)
    {
        return (ell_w + round_words(tile_rows) - 1) / round_words(tile_rows) * round_words(tile_rows);
    }
    static size_t bytes(int ell_w, int tile_rows, bool ffn)
    {
        return off_ent + (size_t)tile_rows * (ell_w > 16 ? row_words(ell_w, tile_rows) : ell_w) * sizeof(uint32_t) +
               (ffn ? (size_t)HR * US * sizeof(T) + (size_t)8 * HR * 32 * sizeof(float) : 0);
    }
};

// W: entries of a neighbour row (8 or 16; 0: any multiple of four, p.ell_w). ONE: one layer
template <typename T, int D, int W, bool FFN, bool ONE>
__global__ __launch_bounds__(HT) void heads_kernel(dg4_heads_args p)
{
    typedef HeadsLds<T, D, W> LDS;
    constexpr int C = D / 32;                     // slices
    constexpr int E = LDS::E;                     // elements in 16 bytes
    constexpr int ROWB = D * (int)sizeof(T);      // bytes of a row
    constexpr int S = ROWB / 64;                  // steps of the matrix cores along a row
    constexpr int UT = E / 4;                     // column tiles of 16 in a unit: 64 bytes of output columns per gate
    constexpr int UC = 16 * UT, CW = 4 * UT;      // columns of a unit, of a lane (16 bytes)
    constexpr int UF = UT * S;                    // fragments of a unit
    constexpr int UD = D / UC;                    // units of D columns
    constexpr int UH = 32 / UC;                   // units of a head's columns
    constexpr int NU = UD > 8 ? UD / 8 : 1;       // units of D columns per wave
    constexpr int LPS = 32 * (int)sizeof(T) / 16; // lanes across a head
    constexpr int YS = LDS::YS, QS = LDS::QS;
    constexpr int WPS = 32 * (int)sizeof(T) / 4;  // 32-bit words of a head's columns
    constexpr int WPR = ROWB / 4;                 // ... of a row
    static_assert(CW == E && 3 * UH <= 8 && (UD <= 8 || UD % 8 == 0), "units");

    extern __shared__ __attribute__((aligned(16))) unsigned char heads_smem[];
    T* resid = (T*)heads_smem;                    // the running state
    T* ybuf = (T*)(heads_smem + LDS::ROWS);       // attention output of all heads, then the normalised rows
    T* qkv = (T*)(heads_smem + LDS::off_qkv);     // this head's Q | K | V of the running state
    float (*stat)[16][HR] = (float (*)[16][HR])(heads_smem + LDS::off_stat);     // [2][unit][row]
    float* att = (float*)(heads_smem + LDS::off_att);            // [part][32] weighted sums, then [part][2] maximum, denominator
    int* ctl = (int*)(heads_smem + LDS::off_ctl); // this tile's and the next one's {first position, rows}, [8] abort word, [12], [13] place in a group
    float* biases = (float*)(ctl + 16);           // [layers][4] of this head
    // Neighbour rows: what is no source (padding, the gate itself) holds relation 0 and the row past the store's end. Narrow
    // rows of one layer lie there as the table has them: they are read once, and rewriting them is on every tile's way to its
    // sources (fp32 / 256, two hops, 30,300 gates: 3.242 -> 3.210 ms). Several layers read them several times (as the table has
    // them: twelve layers fp32 / 128 5.88 -> 5.94 ms; 8300 gates, four layers bf16 / 128 with feed-forward 1274 -> 1289 us), except
    // in bf16 / 256 without feed-forward (four layers 1006 -> 988, three hops 1028 -> 1022, twelve 1381 -> 1375) and, together
    // with lane groups of eight lanes side by side (alone it gains nothing), in fp32 / 128 with feed-forward over rows of 8
    // entries (twelve layers, 9300 gates 5861 -> 5833, four 1768 -> 1764).
    constexpr bool APART = sizeof(T) == 4 && !(W == 8 && FFN && D == 128);
    constexpr bool AS_STORED = W != 0 && (ONE || (sizeof(T) == 2 && D == 256 && !FFN) || (sizeof(T) == 4 && !APART));
    uint32_t* ent = (uint32_t*)(heads_smem + LDS::off_ent);
    const int tile_rows = W ? HR : p.tile_rows;
    const int ell_w = W ? W : LDS::row_words(p.ell_w, tile_rows);
    T* ubuf = (T*)(heads_smem + LDS::off_ent + (size_t)tile_rows * ell_w * sizeof(uint32_t));      // (FFN) the 4D activations
    float* red = (float*)((unsigned char*)ubuf + (size_t)HR * LDS::US * sizeof(T));                // (FFN) [8][16][32] partial sums

    // Lane-derived values, formed anew in every phase (kept across the loops, they and what the compiler derives
    // from them would not fit the registers). Product role of a lane: gate n, columns g*CW .. +CW-1 of a unit.
    int tid, lane, n, g, wave;
    bool qkv_wave, wo_wave;                       // the wave has a unit in the product
    int slice = (int)(blockIdx.x % C);            // (until the workgroup has its seat)
    auto phase = [&](int t) __attribute__((always_inline)) {
        tid = fresh(t); lane = tid & 63; n = lane & 15; g = lane >> 4;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        qkv_wave = wave < 3 * UH; wo_wave = wave < UD;
    };
    phase(threadIdx.x);
    // (what derives from the slice likewise: it is a value like any other once the workgroup has its seat, and kept across
    // the loops its products cost up to 15 scalar registers more in spills, 0.9 % of a two-layer sweep at bf16 / 128)
    auto next_phase = [&]() __attribute__((always_inline)) { phase(tid); __asm__ volatile("" : "+s"(slice)); };
    const int L = ONE ? 1 : p.n_layers;
    const int64_t N = p.n_rows;
    // One layer over wide rows asks for Wo behind the gathers (loads complete in order, and nothing but the gathers is in flight
    // then): with feed-forward, eight hops, 15,300 gates, bf16 / 128 841 -> 828 us, bf16 / 256 1267 -> 1249, fp32 / 256 2257 ->
    // 2225. Not with feed-forward in fp32 / 128 (1074 -> 1082), which takes the form for several layers. In that form a choice at run
    // time is never taken; it costs twelve layers over a partition in bf16 (15,300 gates: hidden 128 5773 -> 5800 us, 256 9954 ->
    // 10,032), but in fp32 / 256 it keeps the early request out of what is scheduled around it (8300 gates 13,520 -> 13,290).
    const bool wo_late = W == 0 && (ONE || (FFN && sizeof(T) == 4 && D == 256 && L == 1));
    uint32_t* flags = p.flags + (int64_t)slice * N;

    // phase timers (DG4_PROFILE): ticket, first projection + wait, attention + exchange, output projection + LayerNorm,
    // next layer's Q|K|V, rows out + K|V, publish, feed-forward
    uint64_t* ticks = (uint64_t*)(heads_smem + LDS::off_ticks);  // eight sums, the last reading
    auto lap = [&](int which) __attribute__((always_inline)) {
        if (p.prof && tid == 0) {
            const uint64_t now = wall_clock64();
            if (which >= 0) ticks[which] += now - ticks[8];
            else for (int i = 0; i < 8; ++i) ticks[i] = 0;
            ticks[8] = now;
        }
    };

    // The fragments of this wave's next unit. Requested through a buffer descriptor (base address and extent in
    // scalar registers, one lane offset for all): a wave without a unit in a product asks with extent 0 and gets
    // zeros without a request, so there is no branch around the loads and no second copy of the registers.
    uint4 ring[UF];
    auto fetch = [&](const void* src, bool active, int bytes) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(src), 0, active ? bytes : 0, 0x00020000);
    };
    auto fill = [&](const void* packed, int group, bool active) __attribute__((always_inline)) {
        const auto rsrc = fetch((const char*)packed + (int64_t)group * (UF * 1024), active, UF * 1024);
#pragma unroll
        for (int f = 0; f < UF; ++f)
            ring[f] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16 + (f & 3) * 1024, (f >> 2) * 4096, 0));
    };
    auto mul = [&](const uint4 (&b)[S], f32x4 (&acc)[UT]) __attribute__((always_inline)) {
#pragma unroll
        for (int nt = 0; nt < UT; ++nt) acc[nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int nt = 0; nt < UT; ++nt) HeadMma<T>::run(ring[nt * S + s], b[s], acc[nt]);
    };
    auto load_rows = [&](const T* buf, uint4 (&b)[S]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < S; ++s) b[s] = *(const uint4*)((const unsigned char*)(buf + n * YS) + s * 64 + g * 16);
    };
    auto cols_of = [&](const f32x4 (&a)[UT], float* t) __attribute__((always_inline)) {
#pragma unroll
        for (int nt = 0; nt < UT; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) t[nt * 4 + i] = a[nt][i];
    };
    // packed weights of layer l, and this wave's unit in each product
    auto wqkv_of = [&](int l) __attribute__((always_inline)) { return (const char*)p.wqkv_packed + (int64_t)l * p.w_layer_stride; };
    auto wo_of = [&](int l) __attribute__((always_inline)) { return (const char*)p.wo_packed + (int64_t)l * p.w_layer_stride; };
    auto fill_qkv = [&](int l) __attribute__((always_inline)) { fill(wqkv_of(l), (wave / UH) * UD + slice * UH + wave % UH, qkv_wave); };
    auto fill_wo = [&](int l) __attribute__((always_inline)) { fill(wo_of(l), wave, wo_wave); };
    // unit u of the K | V of all layers
    const int kv_units = 2 * UH * L;
    auto fill_kv = [&](int u) __attribute__((always_inline)) {
        const int l = u / (2 * UH), part = u % (2 * UH);
        fill(wqkv_of(l), (1 + part / UH) * UD + slice * UH + part % UH, u < kv_units);
    };
    // this wave's part of W2: output columns of this head, S / 2 of the 4*S steps
    constexpr int W2F = UH * UT * S / 2;
    static_assert(W2F <= UF, "the second feed-forward product's fragments fit the ring");
    auto fill_w2 = [&](int l) __attribute__((always_inline)) {
        const char* src = (const char*)p.w2_packed + (int64_t)l * p.ffn_layer_stride;
#pragma unroll
        for (int t = 0; t < UH * UT; ++t) {
            const auto rsrc = fetch(src + ((int64_t)(slice * UH * UT + t) * (4 * S) + wave * (S / 2)) * 1024, true, S / 2 * 1024);
#pragma unroll
            for (int s = 0; s < S / 2; ++s)
                ring[t * (S / 2) + s] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16 + (s & 3) * 1024, (s >> 2) * 4096, 0));
        }
    };
    constexpr int UW1 = 128 / UC;                 // units of this slice's 128 hidden units
    auto fill_w1 = [&](int l) __attribute__((always_inline)) {
        fill((const char*)p.w1_packed + (int64_t)l * p.ffn_layer_stride, slice * UW1 + wave, wave < UW1);
    };

    auto give_up = [&](uint32_t spins) __attribute__((always_inline)) -> bool {
        if (spins > p.spin_limit ||
            ((spins & 63u) == 0 && __hip_atomic_load(&p.ctrl[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
            // the tile is computed from whatever is there (every access stays in bounds), nothing of it is
            // published, and the workgroup leaves after it
            if (lane == 0) {
                __hip_atomic_store(&p.ctrl[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ctl[8] = 1;
            }
            return true;
        }
        return false;
    };
    // exchange words of a tile: [2][tile rows][row] attention outputs, then (FFN) [tile rows][4 rows] activations,
    // [tile rows][D] second products
    constexpr int64_t XA = (int64_t)HR * WPR, XU = (int64_t)HR * 4 * WPR, XY = (int64_t)HR * D;
    constexpr int64_t XT = 2 * XA + (FFN ? XU + XY : 0);
    // NW words per thread, `count` in all, polled until every one carries the tag; take(word index, data)
    auto collect = [&](const uint64_t* src, int count, uint32_t tag, auto nw, auto&& take) __attribute__((always_inline)) {
        constexpr int NW = decltype(nw)::value;
        uint64_t v[NW];
        uint32_t spins = 0;
        // (what has come in is not asked for again: the polls share the memory fabric with the rows being gathered)
        uint32_t missing = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i)
            if (tid + HT * i < count) missing |= 1u << i;
        for (;;) {
#pragma unroll
            for (int i = 0; i < NW; ++i)
                if (missing >> i & 1u) v[i] = __hip_atomic_load(src + tid + HT * i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int i = 0; i < NW; ++i)
                if ((missing >> i & 1u) && (uint32_t)(v[i] >> 32) == tag) missing &= ~(1u << i);
            if (__ballot(missing != 0u) == 0) break;
            __builtin_amdgcn_s_sleep(1);
            if (give_up(++spins)) break;
        }
#pragma unroll
        for (int i = 0; i < NW; ++i)
            if (tid + HT * i < count) take(tid + HT * i, (uint32_t)v[i]);
    };

    uint32_t* sweep_ticket = p.sync + SYNC_TICKET;
    uint64_t* mail = nullptr;                     // the group's [2], by the parity of the tile's number in the group
    auto tile_at = [&](int64_t t) __attribute__((always_inline)) -> uint2 {
        if (!p.pairs) return p.tiles[p.tile_begin + t];
        const uint2 ta = p.tiles[p.tile_begin + 2 * t], tb = p.tiles[p.tile_begin + 2 * t + 1];
        return make_uint2(ta.x, ta.y + tb.y);
    };
    // (one thread) the next ticket of the group, for its `number`-th tile
    auto post_ticket = [&](uint32_t number) __attribute__((always_inline)) {
        int64_t t;
        do t = (int64_t)__hip_atomic_fetch_add(sweep_ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        while (t < p.n_tiles && tile_at(t).y == 0);               // (tables of pairs hold empty tiles)
        put_word(mail + (number & 1), (uint32_t)(t < p.n_tiles ? t : p.n_tiles), number + 1u);
    };
    // (one thread) waits while `blocked()` holds; a wait in which the sweep's tickets still move is none to give up
    auto wait_while = [&](auto&& blocked) __attribute__((always_inline)) {
        dg4_patience patience;
        while (blocked()) {
            __builtin_amdgcn_s_sleep(2);
            if (patience.look(p.spin_limit)) {
                const uint32_t now = __hip_atomic_load(sweep_ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (patience.over(now, p.spin_limit)) __hip_atomic_store(&p.ctrl[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (__hip_atomic_load(&p.ctrl[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) { ctl[8] = 1; return; }
            }
        }
    };
    // (one thread) the group's `number`-th tile, as posted by its first workgroup; rows 0: none left
    auto receive = [&](uint32_t number) __attribute__((always_inline)) {
        uint64_t w = 0;
        wait_while([&]() {
            w = __hip_atomic_load(mail + (number & 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return (uint32_t)(w >> 32) != number + 1u;
        });
        const int64_t t = (uint32_t)(w >> 32) == number + 1u ? (int64_t)(uint32_t)w : p.n_tiles;
        uint2 tile = make_uint2(0, 0);
        if (t < p.n_tiles) tile = tile_at(t);
        ctl[2 * (number & 1)] = (int)tile.x; ctl[2 * (number & 1) + 1] = (int)tile.y;
    };
    // ---- resumed sweeps: K | V of the gates finished before this call, from the caller's embeddings, HR positions
    // at a time, every slice for itself
    auto store_kv = [&](const T* state, int64_t p0, int rows) __attribute__((always_inline)) {
        uint4 b[S];
        f32x4 acc[UT];
        if (wave < kv_units) load_rows(state, b);
#pragma unroll 1
        for (int u = wave; u < kv_units; u += 8) {
            mul(b, acc);
            fill_kv(u + 8);
            const int l = u / (2 * UH), part = u % (2 * UH);
            float v[CW];
            cols_of(acc, v);
            if (n < rows)
                heads_store16((T*)p.kv + (((int64_t)l * C + slice) * N + p0 + n) * 64 + (part / UH) * 32 + (part % UH) * UC + g * CW,
                              Bits16<T>::pack(v));
        }
    };
    // every thread's row stores have completed before the flags go up
    auto publish = [&](int64_t p0, int rows) __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0x0F70);       // vmcnt(0)
        __asm__ volatile("" ::: "memory");
        heads_barrier();
        if (!ctl[8] && tid < rows) __hip_atomic_store(&flags[p0 + tid], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (tid == 0) ctl[8] = 0;
    auto resume_slice = [&](int which) __attribute__((always_inline)) {
        slice = which;
        flags = p.flags + (int64_t)slice * N;
        for (;;) {
            if (tid == 0) ctl[0] = (int)__hip_atomic_fetch_add(&p.sync[slice * 16], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const int64_t t = ctl[0];
            if (t >= p.n_pre) break;
            next_phase();
            const int64_t p0 = t * HR;
            const int rows = (int)(p.pre_rows - p0 < HR ? p.pre_rows - p0 : HR);
            fill_kv(wave);
            for (int piece = tid; piece < rows * (D / E); piece += HT) {
                const int row = piece / (D / E), c = piece % (D / E);
                *(uint4*)&resid[row * YS + c * E] = *((const uint4*)((const T*)p.h_out + (int64_t)p.order[p0 + row] * D) + c);
            }
            heads_barrier();
            store_kv(resid, p0, rows);
            publish(p0, rows);
        }
        __syncthreads();
    };
    // ---- a seat in a group (first the group of the neighbouring workgroups, then any), and the group's first tile.
    // A workgroup that changes its slice leaves no finished gate behind: whoever looks for another group has
    // seen the tickets of every slice run out, and a group by number has one workgroup of every slice.
    int place = -1;                               // group * C + slice; -1: the group was closed; -2: the sweep was given up
    for (int stage = 0; stage < 2; ++stage) {
        if (p.n_pre > 0) {
            const int own = (int)(blockIdx.x % C);
#pragma unroll 1
            for (int i = stage; i < (stage ? C : 1); ++i) resume_slice((own + i) % C);
        }
        if (tid == 0) {
            struct {
                const dg4_heads_args& p; uint32_t* ticket; int* ctl; dg4_patience patience;
                __device__ uint32_t add(uint32_t* q) { return __hip_atomic_fetch_add(q, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
                __device__ uint32_t load(const uint32_t* q) { return __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
                __device__ void store(uint32_t* q, uint32_t v) { __hip_atomic_store(q, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
                __device__ bool cas(uint32_t* q, uint32_t expected, uint32_t v)
                {
                    return __hip_atomic_compare_exchange_strong(q, &expected, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                __device__ void pause() { __builtin_amdgcn_s_sleep(2); }
                __device__ bool leave()           // nothing left, or the sweep was given up
                {
                    const uint32_t drawn = load(ticket);
                    if (drawn >= (uint32_t)p.n_tiles) return true;
                    if (patience.look(p.spin_limit)) {
                        // (a ticket drawn and another workgroup come in are both movements)
                        if (patience.over(drawn + load(p.sync + SYNC_LOOSE), p.spin_limit)) store(&p.ctrl[1], 1u);
                        if (load(&p.ctrl[1])) { ctl[8] = 1; return true; }
                    }
                    return false;
                }
            } mem{p, sweep_ticket, ctl, {}};
            int seat = (int)(blockIdx.x % C);
            uint32_t* word = p.sync + SYNC_GROUP + (int)(blockIdx.x / C) * 16;
            if (stage) {
                const int arrival = (int)mem.add(p.sync + SYNC_LOOSE);
                seat = arrival % C;
                word = p.sync + SYNC_REGROUP + arrival / C * 16;
            }
            // (1024 polls, about a millisecond, at the default limit: workgroups of a launch on an idle device
            // start within some microseconds of each other)
            const dg4_seat at = dg4_sit(mem, word, (uint32_t)C, p.sync + SYNC_FORMED, stage ? 0xFFFFFFFFu : p.spin_limit >> 12);
            ctl[12 + stage] = at.group >= 0 ? at.group * C + seat : ctl[8] ? -2 : -1;
            if (at.group >= 0) {
                mail = (uint64_t*)(p.sync + SYNC_MAIL + at.group * 16);
                if (at.last) post_ticket(0);
                receive(0);
            }
        }
        __syncthreads();
        place = __builtin_amdgcn_readfirstlane(ctl[12 + stage]);
        if (place != -1) break;
    }
    if (place < 0) return;
    slice = place % C;
    const int group = place / C;
    flags = p.flags + (int64_t)slice * N;
    mail = (uint64_t*)(p.sync + SYNC_MAIL + group * 16);
    if (tid < 4 * L) biases[tid] = p.rel_bias[(tid / 4 * C + slice) * 4 + tid % 4];
    lap(-1);
    fill_qkv(0);
    uint64_t* xch = p.exchange + (int64_t)group * XT;
    uint32_t round = 0;                           // layers this group has run: the tag of its exchange words
    for (uint32_t it = 0;; ++it) {
        __syncthreads();                          // the tile; the previous one is done with every buffer
        const int64_t p0 = (uint32_t)ctl[2 * (it & 1)];
        const int rows = ctl[2 * (it & 1) + 1];
        if (rows == 0 || ctl[8]) break;
        lap(0);

        // the gates' rows of x and their neighbour rows
        for (int piece = tid; piece < rows * (D / E); piece += HT) {
            const int row = piece / (D / E), c = piece % (D / E);
            const int64_t id = p.order[p0 + row];
            *(uint4*)&resid[row * YS + c * E] = *((const uint4*)((const T*)p.x + id * D) + c);
        }
        const auto no_source = [&](uint32_t e) __attribute__((always_inline)) { return e == DG4_ELL_PAD || (e >> 30) == 0 ? (uint32_t)N : e; };
        if constexpr (W != 0) {
            for (int i = tid; i < rows * (W / 4); i += HT) {
                const uint4 e = ((const uint4*)(p.ell + p0 * (int64_t)W))[i];
                ((uint4*)ent)[i] = AS_STORED ? e : make_uint4(no_source(e.x), no_source(e.y), no_source(e.z), no_source(e.w));
            }
        } else {
            // entry i of a round lies where lane group i % SG finds its (i / SG)-th: a group reads its eight entries as two
            // 16-byte words, and the groups of a row request ask for entries side by side
            const int row = tid >> p.lanes_log2, lanes = HT / tile_rows, sg_log2 = p.lanes_log2 - (LPS == 4 ? 2 : 3);
            for (int c = tid & (lanes - 1); c < ell_w / 4; c += lanes) {
                uint4 e = make_uint4(DG4_ELL_PAD, DG4_ELL_PAD, DG4_ELL_PAD, DG4_ELL_PAD);
                if (row < rows && 4 * c < p.ell_w) e = *(const uint4*)(p.ell + (p0 + row) * p.ell_w + 4 * c);
                const int i = (4 * c) & ((8 << sg_log2) - 1);
                uint32_t* to = ent + row * ell_w + (4 * c - i) + (i & ((1 << sg_log2) - 1)) * 8 + (i >> sg_log2);
                to[0] = no_source(e.x); to[8] = no_source(e.y); to[16] = no_source(e.z); to[24] = no_source(e.w);
            }
        }
        heads_barrier();

        uint4 b[S];
        f32x4 acc[UT];
        // this head's Q | K | V of the running state
        auto project = [&](const T* rows_of, int l) __attribute__((always_inline)) {
            if (qkv_wave) {
                load_rows(rows_of, b);
                mul(b, acc);
                float v[CW];
                cols_of(acc, v);
                *(uint4*)&qkv[n * QS + (wave / UH) * 32 + (wave % UH) * UC + g * CW] = Bits16<T>::pack(v);
            }
        };
        // Attention roles: SG lane groups of LPS lanes share a gate (a group is a quad of lanes in bfloat16, in fp32 the quads q
        // and q + 2 of 16 lanes). Rows of 8 and 16 entries: group i takes the entries i, i + SG, ...; the K | V
        // are requested a layer ahead (the sources are finished in every layer), so that from the second layer on
        // a narrow row waits for no memory. Wider rows: rounds of eight entries per group, dealt likewise.
        constexpr int SGN = HT / HR / LPS;        // (rows of 8 or 16 entries: tiles of 16)
        constexpr int CH = W ? W / SGN : 8;
        uint4 k4[CH], v4[CH];
        uint32_t en[CH];
        const int lpg = HT / tile_rows, SG = lpg / LPS;           // lanes of a gate: 32 (16 gates) to 256 (2 gates)
        auto gate_of = [&]() __attribute__((always_inline)) { return W ? tid / (HT / HR) : tid >> p.lanes_log2; };
        auto group_of = [&]() __attribute__((always_inline)) {
            const int t = tid & (lpg - 1);
            return LPS == 4 ? t >> 2 : APART ? (t >> 4) * 2 + ((t >> 2) & 1) : t >> 3;
        };
        auto sub_of = [&]() __attribute__((always_inline)) { return LPS == 4 ? tid & 3 : APART ? (tid & 3) | ((tid >> 1) & 4) : tid & 7; };
        auto piece = [&](const uint32_t* at) __attribute__((always_inline)) {
            const uint4 a = ((const uint4*)at)[0], b = ((const uint4*)at)[1];
            en[0] = a.x; en[1] = a.y; en[2] = a.z; en[3] = a.w;
            en[CH - 4] = b.x; en[CH - 3] = b.y; en[CH - 2] = b.z; en[CH - 1] = b.w;
        };
        auto rows_of_layer = [&](int l) __attribute__((always_inline)) {
            return row_buffer((const T*)p.kv + ((int64_t)l * C + slice) * N * 64, 64 * sizeof(T), (uint32_t)N);
        };
        auto is_source = [&](uint32_t e) __attribute__((always_inline)) { return !(AS_STORED && e == DG4_ELL_PAD) && (e >> 30) != 0; };
        // (An entry that is no source asks for the row past the end: zeros, no request. K and V of an entry back to back: they
        // share a cache line, which is gone from the L1 when all K rows of a round are asked for first. Narrow rows have one to
        // four entries per lane group and are left to the compiler: kept apart they cost one layer in bf16 / 128 3 %, 1.463 ->
        // 1.515 ms at 30,300 gates.)
        auto request = [&](int l) __attribute__((always_inline)) {
            const dg4_i32x4 kvb = rows_of_layer(l);
            const uint32_t off = (uint32_t)sub_of() * 16u;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const uint32_t row = AS_STORED && !is_source(en[j]) ? (uint32_t)N : en[j] & 0x3FFFFFFFu;
                k4[j] = row_load16(kvb, row, off);
                v4[j] = row_load16(kvb, row, off + (uint32_t)(32 * sizeof(T)));
                if constexpr (W == 0) __builtin_amdgcn_sched_barrier(0);
            }
        };
        // (W != 0) the sources of a layer
        auto request_first = [&](int l) __attribute__((always_inline)) {
            const int r = gate_of(), grp = group_of();
#pragma unroll
            for (int j = 0; j < CH; ++j) en[j] = r < rows ? ent[r * W + grp + SG * j] : AS_STORED ? DG4_ELL_PAD : (uint32_t)N;
            request(l);
        };
        {
            next_phase();
            project(resid, 0);
            if (!wo_late) fill_wo(0);
            next_phase();
            // ---- the sources of the tile's gates must be published (in this slice)
            {
                const int back = HT - 1 - tid;    // (the waves without a product first)
                const int count = rows * ell_w;
                uint32_t spins = 0;
                int next = back;                  // entries of this thread before `next` have been seen
                for (;;) {
                    bool ok = true;
                    for (; next < count && ok; ) {
                        constexpr int Q = W ? 1 : 4;
                        uint32_t seen[Q];
#pragma unroll
                        for (int q = 0; q < Q; ++q) {
                            const int i = next + HT * q;
                            const uint32_t e = i < count ? ent[i] : 0u;
                            seen[q] = 1u;
                            if (is_source(e)) seen[q] = __hip_atomic_load(flags + (e & 0x3FFFFFFFu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
#pragma unroll
                        for (int q = 0; q < Q; ++q) ok = ok && seen[q] != 0u;
                        if (ok) next += HT * Q;
                    }
                    if (__ballot(!ok) == 0) break;
                    __builtin_amdgcn_s_sleep(1);
                    if (give_up(++spins)) break;
                }
                // (keeps the compiler from moving row loads above the flag loads)
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            heads_barrier();
            lap(1);
            if (W) request_first(0);
#pragma unroll 1
            for (int l = 0; l < L; ++l) {
                const bool last = ONE || l == L - 1;
                // ---- attention with this head: a running maximum, denominator and weighted sum per lane group
                {
                    next_phase();
                    const int r = gate_of(), grp = group_of(), sub = sub_of();
                    const float* bp = biases + 4 * l;
                    const float bias[4] = { bp[0], bp[1], bp[2], bp[3] };
                    const float scale = 0.17677669529663687f;     // 1/sqrt(32)
                    const T* qr = qkv + (r < rows ? r : 0) * QS + sub * E;
                    const uint4 q4 = *(const uint4*)qr;
                    float m = -FLT_MAX, z = 0.f, av[E];
                    {                             // the gate itself (every row holds it), at its running state, in group 0
                        const bool own = r < rows && grp == 0;
                        const float s = fmaf(Bits16<T>::template head_sum<APART>(Bits16<T>::dot(q4, *(const uint4*)(qr + 32))), scale, bias[0]);
                        if (own) { m = fmaxf(s, -FLT_MAX); z = __expf(s - m); }
                        float v[E];
                        Bits16<T>::unpack(*(const uint4*)(qr + 64), v);
#pragma unroll
                        for (int i = 0; i < E; ++i) av[i] = own ? z * v[i] : 0.f;
                    }
                    if constexpr (W != 0) {
                        // One round of SG * CH = W entries. (In bf16 a loop that ends after it, except at hidden 256 without
                        // feed-forward: as straight-line code the round is scheduled together with what stands around it. 10,300
                        // gates: one layer with feed-forward 840 -> 835 us at hidden 128, 1102 -> 1096 at 256, two layers without
                        // 852 -> 847 at 128, but 1170 -> 1172 at 256; fp32 / 256, two layers, 2149 -> 2156.)
                        constexpr bool LOOP = sizeof(T) == 2 && (FFN || D == 128);
                        for (int c0 = grp; !LOOP || c0 < W; c0 += SG * CH) {
                            float sc[CH], cm = m;
#pragma unroll
                            for (int j = 0; j < CH; ++j) {
                                const uint32_t rel = en[j] >> 30;
                                const float dot = Bits16<T>::template head_sum<APART>(Bits16<T>::dot(q4, k4[j]));
                                const float bb = rel == 1 ? bias[1] : rel == 2 ? bias[2] : bias[3];
                                sc[j] = is_source(en[j]) ? fmaf(dot, scale, bb) : -INFINITY;
                                cm = fmaxf(cm, sc[j]);
                            }
                            const float corr = __expf(m - cm);
                            z *= corr;
#pragma unroll
                            for (int i = 0; i < E; ++i) av[i] *= corr;
#pragma unroll
                            for (int j = 0; j < CH; ++j) {
                                const float pj = __expf(sc[j] - cm);  // 0 for what is no source
                                float v[E];
                                Bits16<T>::unpack(v4[j], v);
                                z += pj;
#pragma unroll
                                for (int i = 0; i < E; ++i) av[i] = fmaf(pj, v[i], av[i]);
                            }
                            m = cm;
                            if constexpr (!LOOP) break;
                        }
                    } else {
                        // Eight entries a lane group and round: lane j of a quad ends with the scores of the entries j and j + 4, so
                        // that a score is scaled, masked and exponentiated once and not by every lane of the head, and hands its
                        // weights to the quad: 180 vector instructions a round in fp32, where every lane of a head computing every
                        // score behind a bounds check per entry took 400. Rows of 240 entries: 7.74 -> 7.27 ms with twelve layers at
                        // 15,135 gates in fp32 / 128, 14.1 -> 12.8 at 39,001 with feed-forward in bf16 / 128, 12.5 -> 11.6 with one
                        // layer at 201,024 in bf16 / 256. What is left is the way from the L2 to the registers: 245 KB per compute
                        // unit, layer and tile, 2 us at the 124 GB/s a unit reaches from its L2 with nothing else to do, about 3.5
                        // here. Measured and not kept: the next round's K | V requested under this round's arithmetic (the requests
                        // behind the last round cost what it gains), the first round of the next layer requested during the LayerNorm
                        // (its waves then wait to issue), the next layer's rows touched once per L2.
                        const bool odd = (sub & 1) != 0, upper = (sub & 2) != 0;
                        float zq = 0.f;           // this lane's entries of z
                        const uint32_t* at = ent + r * ell_w + grp * CH;
                        for (int c0 = 0; c0 < ell_w; c0 += SG * CH, at += SG * CH) {
                            piece(at);
                            // rows are padded at the end only: where none of the wave's groups has a source, none follows
                            uint32_t any = 0;
#pragma unroll
                            for (int j = 0; j < CH; ++j) any |= en[j];
                            if (__ballot(any >> 30 != 0) == 0) break;
                            request(l);
                            const uint32_t e0 = at[sub & 3], e1 = at[4 + (sub & 3)];
                            float d[CH];
#pragma unroll
                            for (int j = 0; j < CH; ++j) d[j] = Bits16<T>::dot(q4, k4[j]);
                            const float bb0 = e0 >> 30 == 1 ? bias[1] : e0 >> 30 == 2 ? bias[2] : bias[3];
                            const float bb1 = e1 >> 30 == 1 ? bias[1] : e1 >> 30 == 2 ? bias[2] : bias[3];
                            const float d0 = fmaf(Bits16<T>::quads_sum(quad_sums(d, odd, upper)), scale, bb0);
                            const float d1 = fmaf(Bits16<T>::quads_sum(quad_sums(d + CH - 4, odd, upper)), scale, bb1);
                            const float s0 = is_source(e0) ? d0 : -INFINITY, s1 = is_source(e1) ? d1 : -INFINITY;
                            float cm = fmaxf(s0, s1);
                            cm = fmaxf(cm, xor1(cm));
                            cm = fmaxf(m, fmaxf(cm, xor2(cm)));
                            const float corr = __expf(m - cm), p0 = __expf(s0 - cm), p1 = __expf(s1 - cm);
                            m = cm;
                            z *= corr;
                            zq = fmaf(zq, corr, p0 + p1);
#pragma unroll
                            for (int i = 0; i < E; ++i) av[i] *= corr;
                            const float pj[8] = { of_quad<0>(p0), of_quad<1>(p0), of_quad<2>(p0), of_quad<3>(p0),
                                                  of_quad<0>(p1), of_quad<1>(p1), of_quad<2>(p1), of_quad<3>(p1) };
#pragma unroll
                            for (int j = 0; j < CH; ++j) {
                                float v[E];
                                Bits16<T>::unpack(v4[j], v);
#pragma unroll
                                for (int i = 0; i < E; ++i) av[i] = fmaf(pj[j], v[i], av[i]);
                            }
                        }
                        zq += xor1(zq);
                        z += zq + xor2(zq);
                    }
                    // the groups of a wave that share a gate, merged (all lanes take part)
                    float mm = m;
                    if (LPS == 4) mm = fmaxf(mm, ror<4>(mm));
                    mm = fmaxf(mm, APART ? xor4(mm) : ror<8>(mm));
                    mm = max16(mm);
                    if (tile_rows <= 8) mm = max32(mm);
                    const float f = __expf(m - mm);
                    auto total_of = [&](float x) __attribute__((always_inline)) {
                        x *= f;
                        if (LPS == 4) x += ror<4>(x);
                        x += APART ? xor4(x) : ror<8>(x);
                        x = add16(x);
                        return tile_rows <= 8 ? add32(x) : x;
                    };
                    z = total_of(z);
#pragma unroll
                    for (int i = 0; i < E; ++i) av[i] = total_of(av[i]);
                    const int part = tile_rows == 16 ? r : tid >> 6;      // waves of a gate are consecutive
                    if (grp % (tile_rows == 16 ? 32 / LPS : 64 / LPS) == 0) {
                        *(float4*)&att[part * 32 + sub * E] = make_float4(av[0], av[1], av[2], av[3]);
                        if (E == 8) *(float4*)&att[part * 32 + sub * E + 4] = make_float4(av[E - 4], av[E - 3], av[E - 2], av[E - 1]);
                        if (sub == 0) { att[HR * 32 + 2 * part] = mm; att[HR * 32 + 2 * part + 1] = z; }
                    }
                }
                heads_barrier();
                next_phase();
                // ---- this head's columns go to the other slices ...
                uint64_t* xa = xch + (round & 1u) * XA;
                const uint32_t tag = ++round;     // never 0, the buffer's initial tag
                if (tid < rows * WPS) {
                    const int r = tid / WPS, w = tid % WPS;
                    const int parts = tile_rows >= 8 ? 1 : 8 / tile_rows, first = r * parts;
                    float mm = att[HR * 32 + 2 * first];
                    for (int q = 1; q < parts; ++q) mm = fmaxf(mm, att[HR * 32 + 2 * (first + q)]);
                    float z = 0.f, v0 = 0.f, v1 = 0.f;
                    for (int q = 0; q < parts; ++q) {
                        const float f = __expf(att[HR * 32 + 2 * (first + q)] - mm);
                        z = fmaf(att[HR * 32 + 2 * (first + q) + 1], f, z);
                        const float* vp = att + (first + q) * 32;
                        if (sizeof(T) == 4) v0 = fmaf(vp[w], f, v0);
                        else { v0 = fmaf(vp[2 * w], f, v0); v1 = fmaf(vp[2 * w + 1], f, v1); }
                    }
                    const float rz = 1.0f / z;
                    put_word(xa + (int64_t)r * WPR + slice * WPS + w,
                             sizeof(T) == 4 ? __float_as_uint(v0 * rz) : pack_bf16x2(v0 * rz, v1 * rz), tag);
                }
                if (wo_late) fill_wo(0);
                // ---- ... and theirs come in
                collect(xa, rows * WPR, tag, std::integral_constant<int, HR * WPR / HT>{}, [&](int i, uint32_t data) __attribute__((always_inline)) {
                    *(uint32_t*)((unsigned char*)(ybuf + (i / WPR) * YS) + (i % WPR) * 4) = data;
                });
                heads_barrier();
                lap(2);
                if (last && slice == 0 && tid == HT - 64) post_ticket(it + 1);
                next_phase();
                // ---- s_{l+1} = LN(s_l + a Wo_l), whole rows
                float tv[NU][CW];
                if (wo_wave) {
                    load_rows(ybuf, b);
#pragma unroll
                    for (int u = 0; u < NU; ++u) {
                        mul(b, acc);
                        if (u + 1 < NU) fill(wo_of(l), wave + 8 * (u + 1), true);
                        cols_of(acc, tv[u]);
                    }
                }
                if (FFN) fill_w1(l);
                else if (!last) fill_qkv(l + 1);
                else fill_kv(wave);
                if (W && !ONE && !last) request_first(l + 1);       // the next layer's sources
                next_phase();
                if (p.epilogue) {
                    if (wo_wave) {
#pragma unroll
                        for (int u = 0; u < NU; ++u) {
                            const int unit = wave + 8 * u;
                            float rs[CW], s1 = 0.f;
                            Bits16<T>::unpack(*(const uint4*)&resid[n * YS + unit * UC + g * CW], rs);
#pragma unroll
                            for (int i = 0; i < CW; ++i) { tv[u][i] += rs[i]; s1 += tv[u][i]; }
                            s1 = add32(add16(s1));
                            if (g == 0) stat[0][unit][n] = s1;
                        }
                    }
                    heads_barrier();
                    float mean = 0.f;
                    if (wo_wave) {
#pragma unroll
                        for (int u = 0; u < UD; ++u) mean += stat[0][u][n];
                        mean *= 1.0f / D;
#pragma unroll
                        for (int u = 0; u < NU; ++u) {
                            float s2 = 0.f;
#pragma unroll
                            for (int i = 0; i < CW; ++i) { tv[u][i] -= mean; s2 = fmaf(tv[u][i], tv[u][i], s2); }
                            s2 = add32(add16(s2));
                            if (g == 0) stat[1][wave + 8 * u][n] = s2;
                        }
                    }
                    heads_barrier();
                    if (wo_wave) {
                        float var = 0.f;
#pragma unroll
                        for (int u = 0; u < UD; ++u) var += stat[1][u][n];
                        const float rstd = rsqrtf(var * (1.0f / D) + p.ln_eps);
#pragma unroll
                        for (int u = 0; u < NU; ++u)
#pragma unroll
                            for (int i = 0; i < CW; ++i) tv[u][i] *= rstd;
                    }
                } else {
                    heads_barrier();              // every wave has its operands from ybuf
                }
                if (wo_wave) {
#pragma unroll
                    for (int u = 0; u < NU; ++u) *(uint4*)&ybuf[n * YS + (wave + 8 * u) * UC + g * CW] = Bits16<T>::pack(tv[u]);
                }
                heads_barrier();
                lap(3);
                if constexpr (FFN) {
                    // ---- s_{l+1} <- LN(h + max(h W1, 0) W2), h = ybuf: 128 hidden units here, the others' collected
                    next_phase();
                    uint64_t* xu = xch + 2 * XA;
                    uint64_t* xy = xu + XU;
                    constexpr int US = LDS::US;
                    if (wave < UW1) {
                        load_rows(ybuf, b);
                        mul(b, acc);
                        if (n < rows) {
                            float v[CW];
                            cols_of(acc, v);
#pragma unroll
                            for (int i = 0; i < CW; ++i) v[i] = fmaxf(v[i], 0.f);
                            const uint4 d4 = Bits16<T>::pack(v);
                            uint64_t* dst = xu + (int64_t)n * (4 * WPR) + (slice * 128 + wave * UC + g * CW) * (int)sizeof(T) / 4;
                            put_word(dst, d4.x, tag); put_word(dst + 1, d4.y, tag);
                            put_word(dst + 2, d4.z, tag); put_word(dst + 3, d4.w, tag);
                        }
                    }
                    next_phase();
                    fill_w2(l);
                    // (8 words per thread at a time)
                    for (int i0 = 0; i0 < rows * 4 * WPR; i0 += 8 * HT)
                        collect(xu + i0, rows * 4 * WPR - i0, tag, std::integral_constant<int, 8>{}, [&](int i, uint32_t data) __attribute__((always_inline)) {
                            const int w = i0 + i;
                            *(uint32_t*)((unsigned char*)(ubuf + (w / (4 * WPR)) * US) + (w % (4 * WPR)) * 4) = data;
                        });
                    heads_barrier();
                    next_phase();
                    {
                        f32x4 part[UH * UT];
#pragma unroll
                        for (int t = 0; t < UH * UT; ++t) part[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int s = 0; s < S / 2; ++s) {
                            const uint4 us = *(const uint4*)((const unsigned char*)(ubuf + n * US) + (wave * (S / 2) + s) * 64 + g * 16);
#pragma unroll
                            for (int t = 0; t < UH * UT; ++t) HeadMma<T>::run(ring[t * (S / 2) + s], us, part[t]);
                        }
                        // tile t = (unit t / UT, nt = t % UT): columns (t / UT)*UC + g*CW + (t % UT)*4 + i of the head's 32
#pragma unroll
                        for (int t = 0; t < UH * UT; ++t)
                            *(float4*)&red[(wave * HR + n) * 32 + (t / UT) * UC + g * CW + (t % UT) * 4] =
                                make_float4(part[t][0], part[t][1], part[t][2], part[t][3]);
                    }
                    if (!last) fill_qkv(l + 1);
                    else fill_kv(wave);
                    heads_barrier();
                    next_phase();
                    {
                        const int r = tid / 32, c = tid % 32;
                        if (r < rows) {
                            float y = red[r * 32 + c];
#pragma unroll
                            for (int w = 1; w < 8; ++w) y += red[(w * HR + r) * 32 + c];
                            put_word(xy + (int64_t)r * D + slice * 32 + c, __float_as_uint(y), tag);
                        }
                    }
                    // wave w finishes rows w and w + 8: residual and LayerNorm over the row's D columns
                    constexpr int CPL = D / 64;
#pragma unroll 1
                    for (int r = wave; r < rows; r += 8) {
                        uint64_t v[CPL];
                        uint32_t spins = 0;
                        for (;;) {
                            bool ok = true;
#pragma unroll
                            for (int j = 0; j < CPL; ++j)
                                v[j] = __hip_atomic_load(xy + (int64_t)r * D + j * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                            for (int j = 0; j < CPL; ++j) ok = ok && (uint32_t)(v[j] >> 32) == tag;
                            if (__ballot(!ok) == 0) break;
                            if (give_up(++spins)) break;
                        }
                        float y[CPL], s1 = 0.f;
#pragma unroll
                        for (int j = 0; j < CPL; ++j) {
                            y[j] = __uint_as_float((uint32_t)v[j]) + Elem<T>::load1(ybuf, r * YS + j * 64 + lane);
                            s1 += y[j];
                        }
                        auto wave_sum = [&](float x) __attribute__((always_inline)) {
                            x += ror<8>(x); x += ror<4>(x); x += ror<2>(x); x += ror<1>(x);
                            return add32(add16(x));
                        };
                        const float mean = wave_sum(s1) * (1.0f / D);
                        float s2 = 0.f;
#pragma unroll
                        for (int j = 0; j < CPL; ++j) { y[j] -= mean; s2 = fmaf(y[j], y[j], s2); }
                        const float rstd = rsqrtf(wave_sum(s2) * (1.0f / D) + p.ln_eps);
#pragma unroll
                        for (int j = 0; j < CPL; ++j) Elem<T>::store1(ybuf, r * YS + j * 64 + lane, y[j] * rstd);
                    }
                    heads_barrier();
                    lap(7);
                }
                if (!last) {
                    next_phase();
                    // ---- this head's Q | K | V of the new state
                    project(ybuf, l + 1);
                    fill_wo(l + 1);
                    T* tmp = resid; resid = ybuf; ybuf = tmp;     // the new state is the next layer's residual
                    heads_barrier();
                    lap(4);
                }
            }
            next_phase();
            // ---- the embeddings go out by node id, whole rows dealt over the slices
            for (int piece = tid; piece < rows * (D / E); piece += HT) {
                const int row = piece / (D / E), c = piece % (D / E);
                if (row % C == slice)
                    *((uint4*)((T*)p.h_out + (int64_t)p.order[p0 + row] * D) + c) = *(const uint4*)&ybuf[row * YS + c * E];
            }
        }
        // ---- this head's K | V of every layer from the final embeddings
        next_phase();
        store_kv(ybuf, p0, rows);
        fill_qkv(0);                              // the next tile's first product
        if (tid == HT - 64) receive(it + 1);
        lap(5);
        next_phase();
        publish(p0, rows);
        lap(6);
    }
    if (p.prof && tid == 0)
        for (int i = 0; i < 8; ++i) atomicAdd((unsigned long long*)&p.prof[i], (unsigned long long)ticks[i]);
}

// Everything a sweep starts from: flags, counters and mailboxes down, no tag in the exchange buffer
__global__ void heads_init_kernel(uint32_t* flags, int64_t n_flags, uint32_t* sync, uint32_t* ctrl, uint4* exchange, int64_t n_exchange)
{
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = i0; i < n_flags; i += step) flags[i] = 0u;
    for (int64_t i = i0; i < n_exchange; i += step) exchange[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int64_t i = i0; i < DG4_HEADS_SYNC_BYTES / 4; i += step) sync[i] = 0u;
    if (i0 < 64) ctrl[i0] = 0u;
}

// Weights of all layers into the order the kernel streams them, and the relation biases side by side, in one
// launch. Unit (((group*UT + nt)*steps + s)*64 + lane), 16 bytes, lane = 16*kq + m, holds input rows
// s*4E + kq*E .. +E-1 of column group*16*UT + (m/4)*4*UT + nt*4 + m%4: accumulator register i of lane (n, g) is
// then column group*16*UT + g*4*UT + nt*4 + i, and the lane owns 16 bytes of consecutive columns.
template <typename T>
__global__ __launch_bounds__(256) void heads_pack_kernel(dg4_heads_pack_args p)
{
    constexpr int E = 16 / (int)sizeof(T), UT = E / 4;
    const int d = p.hidden;
    const int64_t per = (int64_t)d * d / E;       // 16-byte units of a [d, d] block
    const int64_t layer_units = per * (p.ffn ? 12 : 4);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int l = (int)(i / layer_units);
    if (l >= p.n_layers) {
        const int64_t j = i - layer_units * p.n_layers;
        const int per_bias = d / 32 * 4;
        if (j < (int64_t)p.n_layers * per_bias) p.bias_all[j] = p.bias[j / per_bias][j % per_bias];
        return;
    }
    int64_t u = i % layer_units;
    const T* w;
    T* out;
    int ld, steps = d / (4 * E);
    if (u < 3 * per) { w = (const T*)p.wqkv[l]; ld = 3 * d; out = (T*)((char*)p.wqkv_packed + l * p.w_layer_stride); }
    else if (u < 4 * per) { u -= 3 * per; w = (const T*)p.wo[l]; ld = d; out = (T*)((char*)p.wo_packed + l * p.w_layer_stride); }
    else if (u < 8 * per) { u -= 4 * per; w = (const T*)p.w1[l]; ld = 4 * d; out = (T*)((char*)p.w1_packed + l * p.ffn_layer_stride); }
    else { u -= 8 * per; w = (const T*)p.w2[l]; ld = d; steps *= 4; out = (T*)((char*)p.w2_packed + l * p.ffn_layer_stride); }
    const int lane = (int)(u & 63), m = lane & 15, kq = lane >> 4;
    const int s = (int)((u >> 6) % steps);
    const int tile = (int)((u >> 6) / steps);
    const int col = (tile / UT) * 16 * UT + (m >> 2) * 4 * UT + (tile % UT) * 4 + (m & 3);
    const int k0 = s * 4 * E + kq * E;
    T v[E];
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = w[(int64_t)(k0 + j) * ld + col];
    *(uint4*)&out[u * E] = *(const uint4*)v;
}

template <typename T, int D>
int launch_heads_t(const dg4_heads_args& a, int64_t groups, hipStream_t s)
{
    constexpr int C = D / 32;
    const bool wide = a.ell_w > 16;
    if (a.ell_w < 8 || a.ell_w % 4 || (!wide && a.ell_w != 8 && a.ell_w != 16)) return hipErrorInvalidValue;
    if (a.tile_rows != 2 && a.tile_rows != 4 && a.tile_rows != 8 && a.tile_rows != 16) return hipErrorInvalidValue;
    if (!wide && a.tile_rows != HR) return hipErrorInvalidValue;
    if (a.n_pre * HR < a.pre_rows || (a.ffn && (!a.w1_packed || !a.w2_packed))) return hipErrorInvalidValue;
    void (*kern)(dg4_heads_args) = nullptr;
    const auto pick = [&](auto w) -> void (*)(dg4_heads_args) {
        constexpr int W = decltype(w)::value;
        // (one layer with feed-forward has a form of its own where that measured ahead: over narrow rows, 19,500 gates, two hops,
        // bf16 / 128 543 -> 535 us, fp32 / 128 718 -> 712, three hops, fp32 / 256 1619 -> 1499; but bf16 / 256 812 -> 820, fp32 / 256
        // over two hops 1472 -> 1476. Over wide rows where the request for Wo stands behind the gathers: fp32 / 256, five hops, 9300
        // gates 1297 -> 1204.)
        if constexpr (W == 0 ? !(sizeof(T) == 4 && D == 128) : D == 128 || (sizeof(T) == 4 && W == 16))
            if (a.ffn && a.n_layers == 1) return heads_kernel<T, D, W, true, true>;
        if (a.ffn) return heads_kernel<T, D, W, true, false>;
        return a.n_layers == 1 ? heads_kernel<T, D, W, false, true> : heads_kernel<T, D, W, false, false>;
    };
    if (a.ell_w == 8) kern = pick(std::integral_constant<int, 8>{});
    else if (a.ell_w == 16) kern = pick(std::integral_constant<int, 16>{});
    else kern = pick(std::integral_constant<int, 0>{});
    const size_t smem = HeadsLds<T, D, 0>::bytes(a.ell_w, a.tile_rows, a.ffn != 0);
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    dg4_heads_args b = a;
    b.lanes_log2 = a.tile_rows == 2 ? 8 : a.tile_rows == 4 ? 7 : a.tile_rows == 8 ? 6 : 5;
    hipLaunchKernelGGL(kern, dim3((unsigned)(groups * C)), dim3(HT), smem, s, b);
    return hipGetLastError();
}

}  // namespace

int64_t dg4_heads_exchange_bytes(int dtype, int hidden, bool ffn, int64_t groups)
{
    const int64_t es = dtype == DG4_F32 ? 4 : 2, wpr = hidden * es / 4;
    return groups * HR * (2 * wpr + (ffn ? 4 * wpr + hidden : 0)) * 8;
}

int dg4_launch_heads_pack(int dtype, const dg4_heads_pack_args& a, hipStream_t s)
{
    const int e = dtype == DG4_F32 ? 4 : 8;
    const int64_t units = (int64_t)a.hidden * a.hidden / e * (a.ffn ? 12 : 4) * a.n_layers + (int64_t)a.n_layers * (a.hidden / 32) * 4;
    const unsigned grid = (unsigned)((units + 255) / 256);
    if (dtype == DG4_F32) hipLaunchKernelGGL(heads_pack_kernel<float>, dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(heads_pack_kernel<uint16_t>, dim3(grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

int dg4_launch_heads(int dtype, int hidden, const dg4_heads_args& a, hipStream_t s)
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return hipErrorInvalidDevice;
    // one workgroup per compute unit, the same number for every slice; only the groups that are launched
    // have exchange words
    const int heads = hidden / 32;
    const int64_t groups = std::max<int64_t>(1, std::min<int64_t>(std::min(cus / heads, dg4_head_groups(heads)), a.n_tiles + a.n_pre));
    const int64_t n_flags = a.n_rows * heads, exchange_bytes = dg4_heads_exchange_bytes(dtype, hidden, a.ffn != 0, groups);
    const int64_t work = std::max<int64_t>(std::max(n_flags, exchange_bytes / 16), DG4_HEADS_SYNC_BYTES / 4);
    hipLaunchKernelGGL(heads_init_kernel, dim3((unsigned)std::min<int64_t>((work + 255) / 256, 2048)), dim3(256), 0, s,
                       a.flags, n_flags, a.sync, a.ctrl, (uint4*)a.exchange, exchange_bytes / 16);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    if (a.n_tiles <= 0) return hipSuccess;
    if (dtype == DG4_F32) return hidden == 128 ? launch_heads_t<float, 128>(a, groups, s) : launch_heads_t<float, 256>(a, groups, s);
    return hidden == 128 ? launch_heads_t<bf16_t, 128>(a, groups, s) : launch_heads_t<bf16_t, 256>(a, groups, s);
}

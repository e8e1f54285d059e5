// Weight compressor, decompressor and dense-twin packer (Fig. 1; Sec. 3.1 Eq. 2; Sec. 3.3 Eq. 6).
// Integer / bit work only: no floating-point instruction touches a weight.
#include "ss_internal.h"
#include "ss_pack_wait.h"
#include <hip/hip_ext.h>
#include <chrono>
#include <thread>

namespace ss {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------------
// header: its words travel as a kernel argument and are written by the packing kernel's first workgroup
// ---------------------------------------------------------------------------------------------
constexpr int kHdrWords = kHdrFirstBad + 1;
struct PackHeader {
    uint32_t w[kHdrWords];
};

static PackHeader pack_header(uint32_t magic, const ss_weight_desc *d, const TileDims &t)
{
    return {{magic, 1u, (uint32_t)d->cout, (uint32_t)d->cin, (uint32_t)d->kh, (uint32_t)d->kw, (uint32_t)d->dtype, (uint32_t)d->korder,
             (uint32_t)t.Mt, (uint32_t)t.Ks, kNoBadBlock}};
}

// ---------------------------------------------------------------------------------------------
// compressor
//
// Lane l of value tile (mt, ks) owns row 32*mt + l%32 and the four blocks 8*ks + {0,1,4,5} + 2*(l/32) of that row, i.e. the
// reduction indices 32*ks + 8*(l/32) + [0,8) and 32*ks + 16 + 8*(l/32) + [0,8): this is where gfx950's 32x32x32 sparse MFMA
// expects the A operand of a lane to come from, given that lane l of the B operand holds the 16 consecutive reduction
// indices 32*ks + 16*(l/32) + [0,16).  (8-bit operands, integer or FP8 -- bytes are copied, never interpreted --: lane l owns
// in slots 2j, 2j+1, j = 0..7, block 16*ks + 8*(j/4) + 4*(l/32) + j%4, because the 32x32x64 instructions pair slot s of
// lane l with the bytes 16*(l/32) + 4*((s%8)/2) + [0,4) of the B lane of the same column in lane group s/8.)
//
// Memory-bound: (2 + 1 + 1.125) bytes per 16-bit weight, 8.125 with an update.  A workgroup packs 32 rows x 32 blocks (128
// weights, kTilesX tiles): consecutive lanes read consecutive blocks of a row (8-byte weight and 4-byte mask loads, 256
// contiguous bytes per row), the packed words cross LDS into tile order and leave as 16-byte stores.  Reading in tile
// order instead (lanes down the rows, 16 contiguous bytes per row and load) touched four times the cache lines:
// 512 x 4608 with an update took 10.5 us so, 6.4 us here (3 TB/s; 3.7 us at the rate of a large copy).
// ---------------------------------------------------------------------------------------------
// binary32 sum of two 16-bit values, rounded to nearest even back to the storage type
template <int DT>
__device__ __forceinline__ uint32_t add16(uint32_t a, uint32_t b)
{
    if constexpr (DT == SS_F16) {
        float s = (float)__builtin_bit_cast(_Float16, (uint16_t)a) + (float)__builtin_bit_cast(_Float16, (uint16_t)b);
        return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)s);
    } else {
        float s = __builtin_bit_cast(float, a << 16) + __builtin_bit_cast(float, b << 16);
        return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)s);
    }
}

constexpr int kPackBlocks = 32;      // blocks of a row per workgroup

// A mask word with exactly two of its four bytes set to one?
__device__ __forceinline__ bool mask_ok(uint32_t m)
{
    return (m & 0xFEFEFEFEu) == 0 && __popc(m) == 2;
}

// The verdict.  The call returns when everything is packed, and it learns that from the last workgroup, which says so in pinned host
// memory: 3 to 5 us sooner than from an event that completes with the kernel (flush of the caches, completion signal, query; profiles/launch_and_packing_waits.md).
// For that, every store here is written through to memory (its acknowledgement then means that every later kernel, copy or host
// access finds it, on whatever stream), every wave waits for its acknowledgements, and every workgroup takes a ticket.  One counter would
// serve 12 ns a ticket (1024 workgroups: 10 us and more), so from kOneCounter workgroups on groups of them count by themselves, each in a cache
// line of its own, and the last of each group counts at the root (0.7 us, the time of 64 tickets).  A counter wraps to zero with its last ticket: nothing has to be reset.
constexpr unsigned kTicketGroups = 16, kOneCounter = 64;
struct __attribute__((aligned(128))) TicketLine {
    unsigned n;
};
__device__ TicketLine ticket_lines[kSlots][kTicketGroups + 1];      // (zero when the library is loaded)

// The workgroup's ticket, taken by one of its threads: true for the last of the `blocks` workgroups.
__device__ __forceinline__ bool last_of_grid(int slot, unsigned blocks)
{
    if (blocks < kOneCounter) return atomicInc(&ticket_lines[slot][0].n, blocks - 1) == blocks - 1;
    const unsigned grp = blockIdx.x % kTicketGroups, in_group = (blocks - grp + kTicketGroups - 1) / kTicketGroups;
    if (atomicInc(&ticket_lines[slot][1 + grp].n, in_group - 1) != in_group - 1) return false;
    return atomicInc(&ticket_lines[slot][0].n, kTicketGroups - 1) == kTicketGroups - 1;
}

// UPD: the weights are first moved to V = W + U (written back over W; every element belongs to exactly one
// thread's blocks), then V is packed.  The place of an invalid block is looked up by find_bad_kernel then.
template <int DT, bool UPD>
__global__ __launch_bounds__(256) void compress_kernel(void *__restrict__ W, const void *__restrict__ U,
                                                       const uint8_t *__restrict__ M, uint8_t *__restrict__ packed,
                                                       int cout, int K, int Mt, int Ks, int Kp, PackHeader hdr, Verdict *verdict, int slot)
{
    constexpr bool BYTES = is_byte_type(DT);
    constexpr int TB = BYTES ? 16 : 8;                    // blocks per row of a tile
    constexpr int TX = kPackBlocks / TB;                  // tiles of the workgroup
    constexpr int J = TB / 2;                             // blocks per lane of a tile
    __shared__ __attribute__((aligned(16))) uint32_t vals[TX * 256];      // the tiles as they will be stored
    __shared__ __attribute__((aligned(16))) uint8_t nibs[TX * 64 * J];    // one nibble per byte, in slot order
    const int tid = threadIdx.x;
    const int G = K >> 2, gx = (Ks + TX - 1) / TX;
    const int mt = blockIdx.x / gx, ks0 = (blockIdx.x - mt * gx) * TX;
    // (all offsets below fit 32 bits: fewer than 2^31 elements, 1.125 bytes each)
    constexpr int kWriteThrough = 17;                     // cache policy sc0 sc1
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(packed, 0, (int)(kHeaderBytes + (unsigned)Mt * (unsigned)Ks * 1024u + (unsigned)Mt * (unsigned)Kp * 256u), 0x00020000);
    if (blockIdx.x == 0 && tid < 64) __builtin_amdgcn_raw_buffer_store_b32(tid < kHdrWords ? hdr.w[tid] : 0u, rp, tid * 4, 0, kWriteThrough);

    const int col = tid & 31;                             // block of the row this thread packs
    const int g = ks0 * TB + col;
    uint32_t m[4];
    uint64_t w[4], u[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int row = mt * 32 + (tid >> 5) + 8 * i;
        m[i] = 0x00000101u;                               // padding: +0 values with the nibble of positions 0, 1
        w[i] = u[i] = 0;
        if (row < cout && g < G) {
            const size_t e = (size_t)row * G + g;         // in blocks
            m[i] = reinterpret_cast<const uint32_t *>(M)[e];
            if constexpr (BYTES) {
                w[i] = static_cast<const uint32_t *>(W)[e];
            } else {
                w[i] = static_cast<const uint64_t *>(W)[e];
                if constexpr (UPD) u[i] = static_cast<const uint64_t *>(U)[e];
            }
        }
    }
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int r = (tid >> 5) + 8 * i, row = mt * 32 + r;
        if constexpr (UPD) {
            uint64_t v = 0;
#pragma unroll
            for (int e = 0; e < 4; e++)
                v |= (uint64_t)add16<DT>((uint32_t)(w[i] >> (16 * e)) & 0xFFFFu, (uint32_t)(u[i] >> (16 * e)) & 0xFFFFu) << (16 * e);
            w[i] = v;
            if (row < cout && g < G) __hip_atomic_store(static_cast<uint64_t *>(W) + (size_t)row * G + g, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        const bool ok = mask_ok(m[i]);
        bad |= !ok;
        const int i0 = ok ? (__ffs(m[i]) - 1) >> 3 : 0, i1 = ok ? (31 - __clz(m[i])) >> 3 : 1;
        const int t = col / TB, gl = col % TB;
        // block gl of the tile's row -> lane group and slot pair
        const int ga = BYTES ? (gl >> 2) & 1 : (gl >> 1) & 1;
        const int j = BYTES ? 4 * (gl >> 3) + (gl & 3) : 2 * (gl >> 2) + (gl & 1);
        const int lane = 32 * ga + r;
        if constexpr (BYTES) {
            const uint32_t pair = ((uint32_t)(w[i] >> (8 * i0)) & 0xFFu) | (((uint32_t)(w[i] >> (8 * i1)) & 0xFFu) << 8);
            reinterpret_cast<uint16_t *>(vals)[(t * 64 + lane) * 8 + j] = (uint16_t)pair;
        } else {
            vals[(t * 64 + lane) * 4 + j] = ((uint32_t)(w[i] >> (16 * i0)) & 0xFFFFu) | (((uint32_t)(w[i] >> (16 * i1)) & 0xFFFFu) << 16);
        }
        nibs[(t * 64 + lane) * J + j] = (uint8_t)(i0 | (i1 << 2));
    }
    __shared__ uint32_t bad_s[4];                         // one per wave
    const bool wave_bad = __any(bad);
    if ((tid & 63) == 0) bad_s[tid >> 6] = wave_bad;
    __syncthreads();
    if (tid == 0 && (bad_s[0] | bad_s[1] | bad_s[2] | bad_s[3])) __hip_atomic_store(&verdict->bad, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    // values: one 16-byte vector per thread and 256-vector pass
#pragma unroll
    for (int v = tid; v < TX * 64; v += 256)
        if (ks0 + (v >> 6) < Ks)
            __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4 *>(vals + v * 4), rp, (int)(kHeaderBytes + (((unsigned)mt * Ks + ks0) * 64 + v) * 16), 0, kWriteThrough);
    // indices: one word per lane and tile (8-bit) or pair of tiles (16-bit; TX is even, so pairs do not straddle workgroups)
    const unsigned meta = kHeaderBytes + (unsigned)Mt * Ks * 1024;
    auto word = [&](int t, int lane) {                    // the nibbles of a lane of a tile
        uint32_t out = 0;
#pragma unroll
        for (int q = 0; q < J / 4; q++) {
            const uint32_t b = *reinterpret_cast<const uint32_t *>(nibs + (t * 64 + lane) * J + 4 * q);
            out |= ((b & 0xFu) | ((b >> 4) & 0xF0u) | ((b >> 8) & 0xF00u) | ((b >> 12) & 0xF000u)) << (16 * q);
        }
        return out;
    };
    if (tid < 128) {
        const int t = tid >> 6, lane = tid & 63;
        if constexpr (BYTES) {
            if (ks0 + t < Ks) __builtin_amdgcn_raw_buffer_store_b32(word(t, lane), rp, (int)(meta + (((unsigned)mt * Ks + ks0 + t) * 64 + lane) * 4), 0, kWriteThrough);
        } else if ((ks0 >> 1) + t < Kp) {
            // (the upper half of an odd last pair: blocks past the row's end, i.e. padding nibbles)
            __builtin_amdgcn_raw_buffer_store_b32(word(2 * t, lane) | (word(2 * t + 1, lane) << 16), rp, (int)(meta + (((unsigned)mt * Kp + (ks0 >> 1) + t) * 64 + lane) * 4), 0, kWriteThrough);
        }
    }
    if (slot < 0) return;                                 // uniform
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wave's stores are in memory
    __syncthreads();
    if (tid == 0 && last_of_grid(slot, (unsigned)(Mt * gx))) __hip_atomic_store(&verdict->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The first (row-major) block with an invalid mask, into the header.  Runs only after a compression found one.
__global__ __launch_bounds__(256) void find_bad_kernel(const uint8_t *__restrict__ M, uint32_t *first_bad, uint32_t blocks)
{
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < blocks && !mask_ok(reinterpret_cast<const uint32_t *>(M)[i])) atomicMin(first_bad, i);
}

// thread per (row, block): inverse permutation, writes 4 elements (8 bytes)
__global__ __launch_bounds__(256) void decompress_kernel(const uint8_t *__restrict__ packed, uint16_t *__restrict__ Wm,
                                                         int cout, int K, int Mt, int Ks, int Kp)
{
    int G = K >> 2;
    int tid = blockIdx.x * 256 + threadIdx.x;
    if (tid >= cout * G) return;
    int g = tid % G, row = tid / G;
    int mt = row >> 5, i = row & 31;
    int ks = g >> 3, gl = g & 7;
    int ga = (gl >> 1) & 1;
    int j = 2 * (gl >> 2) + (gl & 1);
    int lane = 32 * ga + i;
    const uint32_t *vals = reinterpret_cast<const uint32_t *>(packed + kHeaderBytes);
    uint32_t pair = vals[(((size_t)mt * Ks + ks) * 64 + lane) * 4 + j];
    const uint32_t *meta = reinterpret_cast<const uint32_t *>(packed + kHeaderBytes + (size_t)Mt * Ks * 1024);
    uint32_t word = meta[((size_t)mt * Kp + (ks >> 1)) * 64 + lane] >> (16 * (ks & 1));
    uint32_t nib = (word >> (4 * j)) & 0xFu;
    int i0 = nib & 3, i1 = (nib >> 2) & 3;
    uint64_t w64 = 0;
    w64 |= (uint64_t)(pair & 0xFFFFu) << (16 * i0);
    w64 |= (uint64_t)(pair >> 16) << (16 * i1);
    *reinterpret_cast<uint2 *>(Wm + (size_t)row * K + 4 * (size_t)g) = make_uint2((uint32_t)w64, (uint32_t)(w64 >> 32));
}

// thread per (row, block): inverse permutation, writes 4 bytes
__global__ __launch_bounds__(256) void decompress8_kernel(const uint8_t *__restrict__ packed, uint8_t *__restrict__ Wm,
                                                          int cout, int K, int Mt, int Ks)
{
    int G = K >> 2;
    int tid = blockIdx.x * 256 + threadIdx.x;
    if (tid >= cout * G) return;
    int g = tid % G, row = tid / G;
    int mt = row >> 5, i = row & 31;
    int ks = g >> 4, gl = g & 15;
    int ga = (gl >> 2) & 1;
    int j = 4 * (gl >> 3) + (gl & 3);
    int lane = 32 * ga + i;
    const uint16_t *vals = reinterpret_cast<const uint16_t *>(packed + kHeaderBytes);
    uint32_t pair = vals[(((size_t)mt * Ks + ks) * 64 + lane) * 8 + j];
    const uint32_t *meta = reinterpret_cast<const uint32_t *>(packed + kHeaderBytes + (size_t)Mt * Ks * 1024);
    uint32_t nib = (meta[((size_t)mt * Ks + ks) * 64 + lane] >> (4 * j)) & 0xFu;
    int i0 = nib & 3, i1 = (nib >> 2) & 3;
    uint32_t w = ((pair & 0xFFu) << (8 * i0)) | ((pair >> 8) << (8 * i1));
    *reinterpret_cast<uint32_t *>(Wm + (size_t)row * K + 4 * (size_t)g) = w;
}

// Dense twin operand.  16-bit: tile (mt, ks, h), lane l, slot s <-> k = 32*ks + 16*(l/32) + 8*h + s; 8-bit: slot s <->
// k = 64*ks + 32*(l/32) + 16*h + s.  Either way a lane's slots are 16 contiguous bytes of a row, and the 32 rows x 256 bytes
// of a workgroup are 4 reduction steps: consecutive lanes read consecutive pieces of a row, the masked values cross LDS into
// tile order.  Rows are read in units of UB bytes, the largest of 16 .. 1 that divides a row (in elements with their mask
// bytes; UB / element size of them).
template <typename T, int UE>      // T: element; UE: elements per unit
__global__ __launch_bounds__(256) void dense_pack_kernel(const T *__restrict__ W, const uint8_t *__restrict__ M,
                                                         uint8_t *__restrict__ dense, int cout, int K, int Mt, int Ks, PackHeader hdr)
{
    struct __attribute__((aligned(sizeof(T) * UE))) Unit { T e[UE]; };
    struct __attribute__((aligned(UE))) Mask { uint8_t e[UE]; };
    constexpr int STEP = 64 / (int)sizeof(T);             // reduction indices per step (64 bytes)
    constexpr int UNITS = 256 / (int)sizeof(Unit);        // units per row and workgroup
    __shared__ __attribute__((aligned(16))) uint8_t tile[32 * 256];
    const int tid = threadIdx.x, gx = (Ks + 3) / 4;
    const int mt = blockIdx.x / gx, ks0 = (blockIdx.x - mt * gx) * 4;
    if (blockIdx.x == 0 && tid < 64) reinterpret_cast<uint32_t *>(dense)[tid] = tid < kHdrWords ? hdr.w[tid] : 0u;
    for (int i = tid; i < 32 * UNITS; i += 256) {
        const int r = i / UNITS, b = (i % UNITS) * (int)sizeof(Unit);      // row, byte inside the workgroup's 256
        const int row = mt * 32 + r, k = ks0 * STEP + b / (int)sizeof(T);
        Unit v{};
        if (row < cout && k < K) {                        // (a row is a whole number of units)
            v = *reinterpret_cast<const Unit *>(W + (size_t)row * K + k);
            if (M != nullptr) {
                const Mask m = *reinterpret_cast<const Mask *>(M + (size_t)row * K + k);
#pragma unroll
                for (int e = 0; e < UE; e++) v.e[e] = m.e[e] != 0 ? v.e[e] : (T)0;
            }
        }
        // step b/64, lane group (b/32)%2, half (b/16)%2
        *reinterpret_cast<Unit *>(tile + (b >> 6) * 2048 + ((b >> 4) & 1) * 1024 + (32 * ((b >> 5) & 1) + r) * 16 + (b & 15)) = v;
    }
    __syncthreads();
    for (int v = tid; v < 512; v += 256)
        if (ks0 + (v >> 7) < Ks)
            *reinterpret_cast<uint4 *>(dense + kHeaderBytes + (((size_t)mt * Ks + ks0) * 128 + v) * 16) = *reinterpret_cast<const uint4 *>(tile + v * 16);
}

}  // namespace ss

using namespace ss;

extern "C" const char *ss_status_string(int status)
{
    switch (status) {
        case SS_OK: return "SS_OK";
        case SS_ERR_INVALID_ARG: return "SS_ERR_INVALID_ARG: null pointer, bad size or unknown enum";
        case SS_ERR_BAD_MASK: return "SS_ERR_BAD_MASK: a block of 4 mask entries does not hold exactly two ones";
        case SS_ERR_UNSUPPORTED: return "SS_ERR_UNSUPPORTED: K is not a multiple of 4, or sizes exceed the index range";
        case SS_ERR_WORKSPACE: return "SS_ERR_WORKSPACE: workspace too small";
        case SS_ERR_HIP: return "SS_ERR_HIP: a HIP runtime call failed";
        default: return "unknown status";
    }
}

extern "C" int ss_packed_bytes(const ss_weight_desc *desc, size_t *packed_bytes)
{
    if (!packed_bytes) return SS_ERR_INVALID_ARG;
    int st = check_desc(desc, true);
    if (st != SS_OK) return st;
    *packed_bytes = packed_size(tile_dims(desc));
    return SS_OK;
}

extern "C" int ss_dense_bytes(const ss_weight_desc *desc, size_t *dense_bytes)
{
    if (!dense_bytes) return SS_ERR_INVALID_ARG;
    int st = check_desc(desc, false);
    if (st != SS_OK) return st;
    *dense_bytes = dense_size(tile_dims(desc));
    return SS_OK;
}

constexpr int kPollMicroseconds = 1000, kSleepMicroseconds = 50, kSleepsPerQuery = 1000;

// *running: the kernel is on the stream, and this call has not seen its end.
template <int DT, bool UPD>
static int launch_compress(const ss_weight_desc *desc, const TileDims &t, void *W, const void *U, const uint8_t *M, uint8_t *packed,
                           const Waiter &w, hipStream_t s, bool *running)
{
    constexpr int steps = kPackBlocks / (is_byte_type(DT) ? 16 : 8);      // reduction steps per workgroup
    const long long blocks = (long long)t.Mt * ((t.Ks + steps - 1) / steps);
    if (blocks > 0x7FFFFFFFll) return SS_ERR_UNSUPPORTED;
    // (launched by the calls that return their own status: what hipGetLastError says may be an earlier call's)
    int K = t.K, Mt = t.Mt, Ks = t.Ks, Kp = t.Kp, cout = desc->cout, slot = w.slot;
    Verdict *verdict = w.verdict;
    PackHeader hdr = pack_header(kMagicSparse, desc, t);
    void *args[] = {&W, &U, &M, &packed, &cout, &K, &Mt, &Ks, &Kp, &hdr, &verdict, &slot};
    const void *const kernel = reinterpret_cast<const void *>(&compress_kernel<DT, UPD>);
    const dim3 grid((unsigned)blocks), block(256);
    const hipError_t sent = slot < 0 ? hipExtLaunchKernel(kernel, grid, block, args, 0, s, nullptr, w.done, 0) : hipLaunchKernel(kernel, grid, block, args, 0, s);
    const bool earlier = hipGetLastError() != hipSuccess;      // an earlier call's error is reported as everywhere, but behind the wait
    if (sent != hipSuccess) return SS_ERR_HIP;
    *running = true;
    // Polled without a pause for as long as packing itself takes.  A longer wait is for earlier work on the stream, which may take
    // any time: it sleeps between two looks, about 0.1 ms each with the timer's own slack, so the call returns at most that much late.
    // (hipEventSynchronize and hipStreamSynchronize keep the core busy throughout, with hipEventBlockingSync too: behind
    // 300 ms of work 300 ms of processor time, 8 here.)
    const auto since = std::chrono::steady_clock::now();
    hipError_t e = hipSuccess;
    auto pending = [&] {
        if (w.slot >= 0) return __atomic_load_n(&w.verdict->done, __ATOMIC_ACQUIRE) == 0;
        return (e = hipEventQuery(w.done)) == hipErrorNotReady;
    };
    for (int sleeps = 0; pending();) {
        if (std::chrono::steady_clock::now() - since <= std::chrono::microseconds(kPollMicroseconds)) continue;
        std::this_thread::sleep_for(std::chrono::microseconds(kSleepMicroseconds));
        // (now and then: a stream that has failed, or is done and left no verdict, will not leave one)
        if (w.slot >= 0 && ++sleeps % kSleepsPerQuery == 0 && (e = hipStreamQuery(s)) != hipErrorNotReady) {
            if (e == hipSuccess && !pending()) break;
            return SS_ERR_HIP;
        }
    }
    if (e != hipSuccess && e != hipErrorNotReady) return SS_ERR_HIP;
    *running = false;
    return earlier ? SS_ERR_HIP : SS_OK;
}

static int compress_entry(const ss_weight_desc *desc, void *W, const void *U, const uint8_t *M, void *packed,
                          int32_t *bad_row_group, void *stream)
{
    int st = check_desc(desc, true);
    if (st != SS_OK) return st;
    if (!W || !M || !packed) return SS_ERR_INVALID_ARG;
    const bool i8 = is_byte_type(desc->dtype);
    if (i8 && U) return SS_ERR_UNSUPPORTED;       // the update is defined on the 16-bit floats only
    if (!aligned(W, i8 ? 4 : 8) || !aligned(M, 4) || !aligned(packed, 16) || (U && !aligned(U, 8))) return SS_ERR_INVALID_ARG;
    TileDims t = tile_dims(desc);
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t *p = static_cast<uint8_t *>(packed);
    // A call that waits cannot be recorded: under capture the kernel would only run at a replay, and an event that was never
    // recorded reads as complete, so the mask would pass unseen.  Refused before anything is enqueued.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
        (void)hipGetLastError();                          // (reported here, not by the next launch)
        return SS_ERR_HIP;
    }
    if (cap != hipStreamCaptureStatusNone) return SS_ERR_HIP;
    Waiter wt;
    bool running = false;
    if (!take_waiter(&wt)) return SS_ERR_HIP;
    if (i8) st = launch_compress<SS_I8, false>(desc, t, W, nullptr, M, p, wt, s, &running);
    else if (!U) st = launch_compress<SS_F16, false>(desc, t, W, nullptr, M, p, wt, s, &running);
    else if (desc->dtype == SS_F16) st = launch_compress<SS_F16, true>(desc, t, W, U, M, p, wt, s, &running);
    else st = launch_compress<SS_BF16, true>(desc, t, W, U, M, p, wt, s, &running);
    if (st == SS_ERR_HIP && running) return st;           // (the kernel may still run: the waiter is not handed out again)
    const bool bad = __atomic_load_n(&wt.verdict->bad, __ATOMIC_RELAXED) != 0;
    give_waiter(wt);
    if (st != SS_OK || !bad) return st;
    // an invalid mask: find its first block and leave it in the header
    uint32_t first_bad = 0;
    uint32_t *word = reinterpret_cast<uint32_t *>(p) + kHdrFirstBad;
    const uint32_t n = (uint32_t)desc->cout * (uint32_t)t.G;
    find_bad_kernel<<<(n + 255) / 256, 256, 0, s>>>(M, word, n);
    if (hipGetLastError() != hipSuccess) return SS_ERR_HIP;
    if (hipMemcpyAsync(&first_bad, word, 4, hipMemcpyDeviceToHost, s) != hipSuccess) return SS_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return SS_ERR_HIP;
    if (bad_row_group) {
        bad_row_group[0] = (int32_t)(first_bad / (uint32_t)t.G);
        bad_row_group[1] = (int32_t)(first_bad % (uint32_t)t.G);
    }
    return SS_ERR_BAD_MASK;
}

extern "C" int ss_mask_compress(const ss_weight_desc *desc, const void *W, const uint8_t *M, void *packed,
                                int32_t *bad_row_group, void *stream)
{
    return compress_entry(desc, const_cast<void *>(W), nullptr, M, packed, bad_row_group, stream);   // W is only read
}

extern "C" int ss_mask_update_compress(const ss_weight_desc *desc, void *W, const void *U, const uint8_t *M,
                                       void *packed, int32_t *bad_row_group, void *stream)
{
    if (!U) return SS_ERR_INVALID_ARG;
    return compress_entry(desc, W, U, M, packed, bad_row_group, stream);
}

extern "C" int ss_mask_decompress(const ss_weight_desc *desc, const void *packed, void *W_masked_out, void *stream)
{
    int st = check_desc(desc, true);
    if (st != SS_OK) return st;
    if (!packed || !W_masked_out) return SS_ERR_INVALID_ARG;
    const bool i8 = is_byte_type(desc->dtype);
    if (!aligned(packed, 16) || !aligned(W_masked_out, i8 ? 4 : 8)) return SS_ERR_INVALID_ARG;
    TileDims t = tile_dims(desc);
    int total = desc->cout * t.G;
    if (i8) {
        decompress8_kernel<<<(total + 255) / 256, 256, 0, static_cast<hipStream_t>(stream)>>>(
            static_cast<const uint8_t *>(packed), static_cast<uint8_t *>(W_masked_out), desc->cout, t.K, t.Mt, t.Ks);
        return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
    }
    decompress_kernel<<<(total + 255) / 256, 256, 0, static_cast<hipStream_t>(stream)>>>(
        static_cast<const uint8_t *>(packed), static_cast<uint16_t *>(W_masked_out), desc->cout, t.K, t.Mt, t.Ks, t.Kp);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}

extern "C" int ss_weights_check(const ss_weight_desc *desc, const void *weights, int32_t sparse, void *stream)
{
    int st = check_desc(desc, sparse != 0);
    if (st != SS_OK) return st;
    if (!weights || !aligned(weights, 16)) return SS_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint32_t hdr[kHdrFirstBad + 1];
    if (hipMemcpyAsync(hdr, weights, sizeof(hdr), hipMemcpyDeviceToHost, s) != hipSuccess) return SS_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return SS_ERR_HIP;
    const TileDims t = tile_dims(desc);
    const uint32_t want[10] = {sparse ? kMagicSparse : kMagicDense, 1u, (uint32_t)desc->cout, (uint32_t)desc->cin,
                               (uint32_t)desc->kh, (uint32_t)desc->kw, (uint32_t)desc->dtype, (uint32_t)desc->korder,
                               (uint32_t)t.Mt, (uint32_t)t.Ks};
    for (int i = 0; i < 10; i++)
        if (hdr[i] != want[i]) return SS_ERR_INVALID_ARG;
    if (sparse && hdr[kHdrFirstBad] != kNoBadBlock) return SS_ERR_BAD_MASK;
    return SS_OK;
}

extern "C" int ss_dense_pack(const ss_weight_desc *desc, const void *W, const uint8_t *M, void *dense, void *stream)
{
    int st = check_desc(desc, false);
    if (st != SS_OK) return st;
    if (!W || !dense) return SS_ERR_INVALID_ARG;
    if (!aligned(W, is_byte_type(desc->dtype) ? 1 : 2) || !aligned(dense, 16)) return SS_ERR_INVALID_ARG;
    TileDims t = tile_dims(desc);
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t *p = static_cast<uint8_t *>(dense);
    const PackHeader hdr = pack_header(kMagicDense, desc, t);
    const long long blocks = (long long)t.Mt * ((t.Ks + 3) / 4);
    if (blocks > 0x7FFFFFFFll) return SS_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)blocks), block(256);
    // elements per load: as many as divide a row and as W's and M's addresses allow
    auto fits = [&](int elems, int esize) {
        return t.K % elems == 0 && aligned(W, (size_t)elems * esize) && (!M || aligned(M, (size_t)elems));
    };
    if (is_byte_type(desc->dtype)) {
        const uint8_t *w = static_cast<const uint8_t *>(W);
        if (fits(16, 1)) dense_pack_kernel<uint8_t, 16><<<grid, block, 0, s>>>(w, M, p, desc->cout, t.K, t.Mt, t.Ks, hdr);
        else if (fits(4, 1)) dense_pack_kernel<uint8_t, 4><<<grid, block, 0, s>>>(w, M, p, desc->cout, t.K, t.Mt, t.Ks, hdr);
        else dense_pack_kernel<uint8_t, 1><<<grid, block, 0, s>>>(w, M, p, desc->cout, t.K, t.Mt, t.Ks, hdr);
    } else {
        const uint16_t *w = static_cast<const uint16_t *>(W);
        if (fits(8, 2)) dense_pack_kernel<uint16_t, 8><<<grid, block, 0, s>>>(w, M, p, desc->cout, t.K, t.Mt, t.Ks, hdr);
        else if (fits(4, 2)) dense_pack_kernel<uint16_t, 4><<<grid, block, 0, s>>>(w, M, p, desc->cout, t.K, t.Mt, t.Ks, hdr);
        else dense_pack_kernel<uint16_t, 1><<<grid, block, 0, s>>>(w, M, p, desc->cout, t.K, t.Mt, t.Ks, hdr);
    }
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}

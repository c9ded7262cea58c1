/* GENERATED by gen_constants.py -- do not edit.  BLS12-381 Montgomery constants,
 * 32-bit limbs, little-endian limb order.  Fp: R = 2^384; Fr: R = 2^256. */
#pragma once
#include <stdint.h>
namespace tc {
struct FpParams {
    static constexpr int N = 12;
    static constexpr uint32_t INV = 0xfffcfffdu;            /* -mod^-1 mod 2^32 */
    static constexpr uint32_t MOD[12] = {0xffffaaabu, 0xb9feffffu, 0xb153ffffu, 0x1eabfffeu, 0xf6b0f624u, 0x6730d2a0u, 0xf38512bfu, 0x64774b84u, 0x434bacd7u, 0x4b1ba7b6u, 0x397fe69au, 0x1a0111eau};
    static constexpr uint32_t ONE[12] = {0x0002fffdu, 0x76090000u, 0xc40c0002u, 0xebf4000bu, 0x53c758bau, 0x5f489857u, 0x70525745u, 0x77ce5853u, 0xa256ec6du, 0x5c071a97u, 0xfa80e493u, 0x15f65ec3u};   /* R mod q */
    static constexpr uint32_t R2[12] = {0x1c341746u, 0xf4df1f34u, 0x09d104f1u, 0x0a76e6a6u, 0x4c95b6d5u, 0x8de5476cu, 0x939d83c0u, 0x67eb88a9u, 0xb519952du, 0x9a793e85u, 0x92cae3aau, 0x11988fe5u};    /* R^2 mod q */
    static constexpr uint32_t R3[12] = {0xd94ca1e0u, 0xed48ac6bu, 0x03a7adf8u, 0x315f831eu, 0x615e29ddu, 0x9a53352au, 0x921e1761u, 0x34c04e5eu, 0x65724728u, 0x2512d435u, 0x91755d4du, 0x0aa63460u};    /* R^3 mod q */
    static constexpr uint32_t MOD_M2[12] = {0xffffaaa9u, 0xb9feffffu, 0xb153ffffu, 0x1eabfffeu, 0xf6b0f624u, 0x6730d2a0u, 0xf38512bfu, 0x64774b84u, 0x434bacd7u, 0x4b1ba7b6u, 0x397fe69au, 0x1a0111eau}; /* q - 2 */
    static constexpr int GCD_ROUNDS = 27;              /* ceil((2 len(q) - 1) / 30) + 1 */
    static constexpr uint32_t GCD_FIX[12] = {0x317468b8u, 0x0a55fea2u, 0x933216c5u, 0x9941e988u, 0xe6642962u, 0x63286e14u, 0xb0bd8ff3u, 0x9968153eu, 0x87cd505fu, 0x328225ebu, 0x80d97151u, 0x0c9d232eu}; /* 4^GCD_ROUNDS * R^3 mod q */
    static constexpr uint32_t HALF[12] = {0xffffd555u, 0xdcff7fffu, 0x58a9ffffu, 0x0f55ffffu, 0x7b587b12u, 0xb3986950u, 0x79c2895fu, 0xb23ba5c2u, 0x21a5d66bu, 0x258dd3dbu, 0x1cbff34du, 0x0d0088f5u};  /* (q - 1) / 2 */
};
struct FrParams {
    static constexpr int N = 8;
    static constexpr uint32_t INV = 0xffffffffu;            /* -mod^-1 mod 2^32 */
    static constexpr uint32_t MOD[8] = {0x00000001u, 0xffffffffu, 0xfffe5bfeu, 0x53bda402u, 0x09a1d805u, 0x3339d808u, 0x299d7d48u, 0x73eda753u};
    static constexpr uint32_t ONE[8] = {0xfffffffeu, 0x00000001u, 0x00034802u, 0x5884b7fau, 0xecbc4ff5u, 0x998c4fefu, 0xacc5056fu, 0x1824b159u};   /* R mod q */
    static constexpr uint32_t R2[8] = {0xf3f29c6du, 0xc999e990u, 0x87925c23u, 0x2b6cedcbu, 0x7254398fu, 0x05d31496u, 0x9f59ff11u, 0x0748d9d9u};    /* R^2 mod q */
    static constexpr uint32_t R3[8] = {0x439b73afu, 0xc62c1807u, 0x8cf06990u, 0x1b3e0d18u, 0xc7b5f418u, 0x73d13c71u, 0xc8db33e9u, 0x6e2a5bb9u};    /* R^3 mod q */
    static constexpr uint32_t MOD_M2[8] = {0xffffffffu, 0xfffffffeu, 0xfffe5bfeu, 0x53bda402u, 0x09a1d805u, 0x3339d808u, 0x299d7d48u, 0x73eda753u}; /* q - 2 */
    static constexpr int GCD_ROUNDS = 18;              /* ceil((2 len(q) - 1) / 30) + 1 */
    static constexpr uint32_t GCD_FIX[8] = {0xcb9d63b7u, 0x6e19d729u, 0x5f8be0ccu, 0xf8f3f232u, 0xa5edc8e5u, 0xbab78932u, 0xc66409cfu, 0x4a73978cu}; /* 4^GCD_ROUNDS * R^3 mod q */
    static constexpr uint32_t HALF[8] = {0x80000000u, 0x7fffffffu, 0x7fff2dffu, 0xa9ded201u, 0x04d0ec02u, 0x199cec04u, 0x94cebea4u, 0x39f6d3a9u};  /* (q - 1) / 2 */
    static constexpr int32_t NEG29[9] = {-1, -536870904, -529989567, -457704959, -494949691, -201589968, -354471143, -174404527, -7597479};      /* the 29-bit limbs of q, negated (the lowest is 1) */
    static constexpr int TWO_ADICITY = 32;
    static constexpr uint32_t ROOT[8] = {0x0c17f47cu, 0x9cab6d5cu, 0xfd4b71e5u, 0x1ce1e93du, 0x471dd505u, 0x0d6db230u, 0x743a3b6au, 0x3f0ee990u};  /* a root of unity of order 2^TWO_ADICITY, Montgomery form */
};
struct Fp28Params {
    static constexpr int N = 14;
    static constexpr int32_t NINV = 0xffcfffd;              /* -p^-1 mod 2^28 */
    static constexpr int32_t PINV = 0x0030003;              /* p^-1 mod 2^28 */
    static constexpr int32_t MOD[14] = {0xfffaaab, 0xfefffff, 0x3ffffb9, 0xfffeb15, 0x6241eab, 0xa0f6b0f, 0xf6730d2, 0xf38512b, 0x4774b84, 0x4bacd76, 0xba7b643, 0xe69a4b1, 0x1ea397f, 0x001a011};
    static constexpr int32_t ONE[14] = {0x347fcb8, 0xd800000, 0x002b119, 0x0cde6d2, 0xc7212e0, 0x83a2090, 0x037669f, 0xda0f73e, 0x9b09b42, 0x1297bb0, 0x515d98f, 0x012ca7c, 0x659fcfa, 0x000577a};   /* 2^392 mod p */
    static constexpr int GCD_ROUNDS = 29;                /* ceil((2 len(p) - 1) / 28) + 1 rounds of 28 steps */
    static constexpr int32_t INV_FIX[14] = {0x4d1dd0e, 0x41d94cc, 0x109f399, 0x8cb551c, 0x2b7ff56, 0x980df0c, 0x71cc8ea, 0x76862c6, 0xbf76e0c, 0xae37e1d, 0x527bf47, 0xb194cef, 0x04d56b3, 0x0008347};  /* 2^1168 mod p: 1 / a (mod p) -> the 28-bit form of R^2 / a, R = 2^384 */
    static constexpr int32_t INV_START[14] = {0x10370ed, 0x6d1c345, 0xe243d62, 0xec45c53, 0x3b1d65a, 0x093317d, 0xb4f36a0, 0x5d74088, 0xc10ea72, 0x865d118, 0x7320a75, 0xfd5cd50, 0xcc8a759, 0x000c8d4};  /* 2^784 mod p: a R -> R / a under the radix R = 2^392 */
    static constexpr int32_t INV_SCALE[14] = {0x1f7b890, 0x294cc4d, 0x9f3af22, 0xb5ba56c, 0xcb5c0cc, 0xc0d975c, 0xc89a8c5, 0x6c968b4, 0x22672ea, 0x91de8c9, 0x35652a6, 0x84977c8, 0x424bbb9, 0x00141ab};  /* 2^1176 mod p: a plain 1 / a -> R^2 / a, R = 2^392 */
};
struct Fp30Params {
    static constexpr int32_t NINV = 1073545213;              /* -p^-1 mod 2^30 */
    static constexpr int32_t PINV = 196611;              /* p^-1 mod 2^30 */
    static constexpr int32_t MOD[13] = {-21845, -402915328, 356515836, -352321620, -252304353, 55215067, 288093811, 316751073, -321428361, 517541167, -375082566, -91332614, 1704210};
    static constexpr int32_t ONE[13] = {13762350, 433586176, -192935228, -301937177, 37952645, -425753694, -36732706, 162803105, -437337492, 366579475, 78814996, -442511456, 89578};   /* 2^390 mod p */
};
#define TC_WAVE28_ROWS \
    {0x002faabbu, 0x04c203d2u, 0x02c07e7au, 0x018f8f15u, 0x06c7b6b8u, 0x0961f5b3u, 0x0e3a59f5u, 0x0f43940du, 0x0de40cc3u, 0x0ef9c7a5u, 0x025598bbu, 0x0c2b4463u, 0x01b1fd61u, 0x00019fc3u, 0, 0}, /* (c p + 1) / 2^28, c = -1 / p mod 2^28 */ \
    {0x0fffaaabu, 0x0fefffffu, 0x03ffffb9u, 0x0fffeb15u, 0x06241eabu, 0x0a0f6b0fu, 0x0f6730d2u, 0x0f38512bu, 0x04774b84u, 0x04bacd76u, 0x0ba7b643u, 0x0e69a4b1u, 0x01ea397fu, 0x0001a011u, 0, 0}, /* p */ \
    {0x4fd55580u, 0x47fffffbu, 0x4fffdcfbu, 0x4ff58a9bu, 0x420f55fbu, 0x47b587adu, 0x4398694cu, 0x4c2895f7u, 0x4ba5c275u, 0x4d66bb1fu, 0x43db21a1u, 0x44d258d9u, 0x451cbfefu, 0x00d0088bu, 0, 0}, /* 128 p in raised limbs */ \
    {0x4f555600u, 0x4ffffffbu, 0x4fff73f9u, 0x4fd62a7bu, 0x483d57fbu, 0x4ed61ec0u, 0x4e61a53du, 0x40a257e8u, 0x4e9709e3u, 0x459aec8au, 0x4f6c8693u, 0x43496370u, 0x4472ffc9u, 0x03402239u, 0, 0}, /* 512 p in raised limbs */ \
    {0x0347fcb8u, 0x0d800000u, 0x0002b119u, 0x00cde6d2u, 0x0c7212e0u, 0x083a2090u, 0x0037669fu, 0x0da0f73eu, 0x09b09b42u, 0x01297bb0u, 0x0515d98fu, 0x0012ca7cu, 0x0659fcfau, 0x0000577au, 0, 0}, /* 2^392 mod p */ \
    {0x0450f071u, 0x0cc341c3u, 0x00f2242du, 0x0a6ebfb4u, 0x0ea1bcaau, 0x085e0207u, 0x05294915u, 0x00c96153u, 0x06eaa0bbu, 0x0715fd90u, 0x0e2f899fu, 0x0d455b78u, 0x0a49ef74u, 0x00005d6cu, 0, 0}, /* 2^776 mod p: plain value moved up by 8 bits -> the form */ \
    {0x00000100u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0, 0}, /* 2^8: the form -> plain value moved up by 8 bits */ \
    {0x02421b59u, 0x0bee4867u, 0x01d31002u, 0x04760184u, 0x04cc5086u, 0x0c76dc00u, 0x0aae891bu, 0x0ac70ad2u, 0x0fe377c4u, 0x0e4686b8u, 0x05ed1568u, 0x08f5a180u, 0x002b5c1fu, 0x0000d1a4u, 0, 0} /* beta 2^392 mod p */
/* G1 generator, Montgomery form */
static constexpr uint32_t G1_GEN_X[12] = {0xfd530c16u, 0x5cb38790u, 0x9976fff5u, 0x7817fc67u, 0x143ba1c1u, 0x154f95c7u, 0xf3d0e747u, 0xf0ae6acdu, 0x21dbf440u, 0xedce6eccu, 0x9e0bfb75u, 0x12017741u};
static constexpr uint32_t G1_GEN_Y[12] = {0x0ce72271u, 0xbaac93d5u, 0x7918fd8eu, 0x8c22631au, 0x570725ceu, 0xdd595f13u, 0x50405194u, 0x51ac5829u, 0xad0059c0u, 0x0e1c8c3fu, 0x5008a26au, 0x0bbc3efcu};
/* endomorphism (x, y) -> (beta x, y) = [lambda](x, y), lambda = z^2 - 1 < 2^128 */
static constexpr uint32_t GLV_LAMBDA[4] = {0xffffffffu, 0x00000000u, 0x0001a402u, 0xac45a401u};
static constexpr uint32_t GLV_BETA[12] = {0x8671f071u, 0xcd03c9e4u, 0x1fcda5d2u, 0x5dab2246u, 0xd3851b95u, 0x587042afu, 0x01bacb9eu, 0x8eb60ebeu, 0x83d050d2u, 0x03f97d6eu, 0x54638741u, 0x18f02065u};      /* Montgomery form */
/* pairing (host side): G2 generator on the twist, Montgomery form, (c0, c1) of x then of y */
static constexpr uint32_t G2_GEN[4][12] = {{0x02940a10u, 0xf5f28fa2u, 0x87b4961au, 0xb3f5fb26u, 0x3e2ae580u, 0xa1a893b5u, 0x1a3caee9u, 0x9894999du, 0x1863366bu, 0x6f67b763u, 0x4350bcd7u, 0x05819192u}, {0x9e23f606u, 0xa5a9c075u, 0xbccd60c3u, 0xaaa0c59du, 0xe2867806u, 0x3bb17e18u, 0x8541b367u, 0x1b1ab6ccu, 0xf2158547u, 0xc2b6ed0eu, 0x7360edf3u, 0x11922a09u}, {0x60494c4au, 0x4c730af8u, 0x5e369c5au, 0x597cfa1fu, 0xaa0a635au, 0xe7e6856cu, 0x6e0d495fu, 0xbbefb5e9u, 0xf0ef25a2u, 0x07d3a975u, 0x7e80dae5u, 0x0083fd8eu}, {0xdf64b05du, 0xadc0fc92u, 0x2b1461dcu, 0x18aa270au, 0x3be4eba0u, 0x86adac6au, 0xc93da33au, 0x79495c4eu, 0xa43ccaedu, 0xe7175850u, 0x63de1bf2u, 0x0b2bc2a1u}};
/* (u + 1)^((p - 1) / 6), Montgomery form (c0, c1) */
static constexpr uint32_t FROB1_GAMMA[2][12] = {{0xb319d465u, 0x07089552u, 0xb50a8313u, 0xc6695f92u, 0xd117228fu, 0x97e83cccu, 0xb2dc29eeu, 0xa35baecau, 0x5daace4du, 0x1ce393eau, 0xb0fb66ebu, 0x08f2220fu}, {0x4ce5d646u, 0xb2f66aadu, 0xfc497cecu, 0x5842a06bu, 0x2599d394u, 0xcf4895d4u, 0x40a8e8d0u, 0xc11b9cbau, 0xe5a0de89u, 0x2e3813cbu, 0x88847fafu, 0x110eefdau}};
/* (u + 1)^((p^2 - 1) / 6), Montgomery form (c0, c1) */
static constexpr uint32_t FROB2_GAMMA[2][12] = {{0x798dba3au, 0xecfb361bu, 0x91865a2cu, 0xc100ddb8u, 0x232bda8eu, 0x0ec08ff1u, 0xf1ca4721u, 0xd5c13cc6u, 0xbf7b5c04u, 0x47222a47u, 0xe51c5f59u, 0x0110f184u}, {0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u, 0x00000000u}};
/* |z|, the loop length of the Miller function */
static constexpr uint64_t BLS_Z_ABS = 0xd201000000010000ull;
/* (p^4 - p^2 + 1) / r, 1268 bits */
static constexpr int HARD_EXP_LIMBS = 40;
static constexpr uint32_t HARD_EXP[40] = {0x38e3ba79u, 0xe516c3f4u, 0xe208ccf1u, 0xfa9912aau, 0x335d5b68u, 0x905ce937u, 0xb0dea236u, 0xc71a2629u, 0x996754c8u, 0x83774940u, 0xb6a1e799u, 0x21d160aeu, 0xed237db4u, 0x2ed0b283u, 0x6c6f1821u, 0x915c97f3u, 0xde783765u, 0x67f17fcbu, 0x9096d1b7u, 0x2378b903u, 0x1bdc51dcu, 0x7988f876u, 0x03fc77a1u, 0x20769950u, 0xa621315bu, 0x827eca0bu, 0x8d63cb9fu, 0xe5a72bceu, 0xc28b6f8au, 0xf68f7764u, 0xcf081517u, 0x2f230063u, 0x528d6a9au, 0x94506632u, 0xeb996ca3u, 0xd3cde88eu, 0x195c899eu, 0xc0bd38c3u, 0x3d807d01u, 0x000f686bu};
}  // namespace tc

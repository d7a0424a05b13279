// Positive Gauss-Hermite nodes (roots of He_Q, ascending) of the node counts that the kernels
// are compiled for, as gauss_hermite finds them (Jacobi eigenvalues refined by Newton's
// method): the two ends of the last rounding are both roots to FP64, and every stored state
// and FP32 run follows its bits.
#pragma once

namespace elb {

struct NodeTable {
    int q;
    const double *positive;  // q / 2 values
};

constexpr double kNodes8[] = {
    0x1.140244df60425p-1, 0x1.a2f2e9768a3f2p+0, 0x1.66b7db50ddbecp+1, 0x1.094042d748ee4p+2,
};
constexpr double kNodes12[] = {
    0x1.c711949e60908p-2, 0x1.5722d43422c04p+0, 0x1.21362191c2f29p+1, 0x1.9ca2860f2e400p+1,
    0x1.1165983dc4e75p+2, 0x1.600ec605ccc6dp+2,
};
constexpr double kNodes16[] = {
    0x1.8c0af8ced8268p-2, 0x1.29f0b43504447p+0, 0x1.f3b4fbe349534p+0, 0x1.614fb5b04289ap+1,
    0x1.cce96d4a6c430p+1, 0x1.1f8c9465ada5ap+2, 0x1.5e38f22ad8822p+2, 0x1.a8604ef376e7ap+2,
};
constexpr double kNodes20[] = {
    0x1.634a926e31cc3p-2, 0x1.0afe77649f856p+0, 0x1.bec88746540b2p+0, 0x1.3ab57d3cecdfdp+1,
    0x1.9831a333c7332p+1, 0x1.f8d3ec11c84fep+1, 0x1.2f03616d7eb60p+2, 0x1.650a0e7d0f317p+2,
    0x1.a0ad8256821f2p+2, 0x1.e79e7dc649aaep+2,
};
constexpr double kNodes24[] = {
    0x1.44fcaaa701e6fp-2, 0x1.e826eb1490d09p-1, 0x1.97ee555ce0a70p+0, 0x1.1ec7a68b60b2cp+1,
    0x1.72e8c5ada9cd8p+1, 0x1.c8df0b468b342p+1, 0x1.10aa1ffefe67ap+2, 0x1.3e983ad98d6f2p+2,
    0x1.6ee554687c2dbp+2, 0x1.a2aacda3fd64ap+2, 0x1.dc06669272595p+2, 0x1.103fed2a77985p+3,
};
constexpr double kNodes32[] = {
    0x1.1a28d72c7eea3p-2, 0x1.a791e30c6acd6p-1, 0x1.6187eb184c23ep+0, 0x1.f02116ea70426p+0,
    0x1.3ffac54e39766p+1, 0x1.88b8a7394f347p+1, 0x1.d2883126a7f59p+1, 0x1.0ed96f11da5cap+2,
    0x1.354964dc18905p+2, 0x1.5ccd585c14c3bp+2, 0x1.85b1975b7fcd2p+2, 0x1.b0612bb4cd77fp+2,
    0x1.dd7d05b3d953dp+2, 0x1.0708049ea9d49p+3, 0x1.220f8eeefb5c9p+3, 0x1.427a3f1db919fp+3,
};
constexpr double kNodes40[] = {
    0x1.f983867ff4e0ep-3, 0x1.7b53685f55703p-1, 0x1.3c6c97ed6bf48p+0, 0x1.bbabd32fc4c0ep+0,
    0x1.1dce54b44df01p+1, 0x1.5e3c132cabb4fp+1, 0x1.9f3e4cb2c73c0p+1, 0x1.e0f7b7ffb4979p+1,
    0x1.11c7e75be34a0p+2, 0x1.339a35984e84dp+2, 0x1.560e03ffd90aap+2, 0x1.79447f05ffdf7p+2,
    0x1.9d67314f6f5e8p+2, 0x1.c2abd790ad34ep+2, 0x1.e95abf4324367p+2, 0x1.08ed14e30495ep+3,
    0x1.1e62575a686a8p+3, 0x1.358dc614ffd0dp+3, 0x1.4f68f1a36f0c4p+3, 0x1.6e82123f45da1p+3,
};
constexpr double kNodes48[] = {
    0x1.cdf0dddea679ap-3, 0x1.5a93b43a58422p-1, 0x1.210463c364b44p+0, 0x1.950da2d47302bp+0,
    0x1.04c34ea5c9306p+1, 0x1.3f48fb780231cp+1, 0x1.7a2a42b1c7f3dp+1, 0x1.b57aff0c6c2adp+1,
    0x1.f150e4432c914p+1, 0x1.16e200af886eep+2, 0x1.3577b31b3ac77p+2, 0x1.5478fd57cc5fdp+2,
    0x1.73f7cecbe239bp+2, 0x1.94095665785c1p+2, 0x1.b4c716554d428p+2, 0x1.d6507467fef3ep+2,
    0x1.f8cd156e402d1p+2, 0x1.0e384a3530977p+3, 0x1.20c059b78fd4cp+3, 0x1.3430372e1ebe2p+3,
    0x1.48d2e002762b3p+3, 0x1.5f25480d3f65bp+3, 0x1.781a09b7963d1p+3, 0x1.962d2829d1392p+3,
};
constexpr double kNodes64[] = {
    0x1.9090eb32c613bp-3, 0x1.2c7be7c95c5a8p-1, 0x1.f5015912c23d3p-1, 0x1.5ee9bb54f5139p+0,
    0x1.c388e15869b4bp+0, 0x1.14372701b9b28p+1, 0x1.46d5618874c9bp+1, 0x1.79a7de0349920p+1,
    0x1.acb7cd35cc13ap+1, 0x1.e00eec0c5356ap+1, 0x1.09dbd05708f8fp+2, 0x1.23de8e4908bbap+2,
    0x1.3e15c280f9768p+2, 0x1.588811f385f89p+2, 0x1.733cd1aefd2d1p+2, 0x1.8e3c2bb7e18b2p+2,
    0x1.a98f4d4bfc63ap+2, 0x1.c540a1d1d2e20p+2, 0x1.e15c1f271f8cbp+2, 0x1.fdefaa3402d14p+2,
    0x1.0d85cf130b8e5p+3, 0x1.1c61c336e93bap+3, 0x1.2b9792a6e17c0p+3, 0x1.3b35f8ff64513p+3,
    0x1.4b4facbc38c34p+3, 0x1.5bfd262ab1b8dp+3, 0x1.6d5f95b04e7c3p+3, 0x1.7fa6301832504p+3,
    0x1.931898a880454p+3, 0x1.a82e478fa878ep+3, 0x1.bfcf41c126eb4p+3, 0x1.dc5ba30af9f65p+3,
};
constexpr double kNodes96[] = {
    0x1.477b82ea9a641p-3, 0x1.eb4460a929b20p-2, 0x1.99762f4457d05p-1, 0x1.1eb306bfd1027p+0,
    0x1.70be89e1b9271p+0, 0x1.c2e356ebbf1b8p+0, 0x1.0a939d4b7a3ffp+1, 0x1.33c80eff38663p+1,
    0x1.5d12063c9566bp+1, 0x1.86749ce94edd4p+1, 0x1.aff3047b0a91ep+1, 0x1.d99089918cb7fp+1,
    0x1.01a84bf12cfecp+2, 0x1.169b5f424ff9cp+2, 0x1.2ba35a5759c41p+2, 0x1.40c22f7cbe62bp+2,
    0x1.55f9eaa0f2971p+2, 0x1.6b4cb4a281206p+2, 0x1.80bcd70cbeea6p+2, 0x1.964cc057fdf57p+2,
    0x1.abff08c6aedafp+2, 0x1.c1d677feaad19p+2, 0x1.d7d60b85466dep+2, 0x1.ee00fe4e5684cp+2,
    0x1.022d68cd5b29cp+3, 0x1.0d73abb991ee3p+3, 0x1.18d55f90ee338p+3, 0x1.2454d2152adacp+3,
    0x1.2ff49032df676p+3, 0x1.3bb7711084d0cp+3, 0x1.47a0a3b262581p+3, 0x1.53b3bffd1a522p+3,
    0x1.5ff4dc2df034fp+3, 0x1.6c68a851d8eecp+3, 0x1.791491eff7550p+3, 0x1.85fef324d710fp+3,
    0x1.932f520f9238cp+3, 0x1.a0aeb8216d118p+3, 0x1.ae882d6f8ea0ep+3, 0x1.bcc96c3a0c7e5p+3,
    0x1.cb83efe6826d4p+3, 0x1.dacea06e5d5d9p+3, 0x1.eac89aa19e91bp+3, 0x1.fb9e29c53d7fap+3,
    0x1.06c9471cf74d6p+4, 0x1.108af92fde220p+4, 0x1.1b810e953fc87p+4, 0x1.28c8bd9f31502p+4,
};
constexpr double kNodes200[] = {
    0x1.c66250ad522abp-4, 0x1.54cb857a9b89cp-2, 0x1.1c01e9088e455p-1, 0x1.8da286aae6125p-1,
    0x1.ff496641cb7c8p-1, 0x1.387c29d9863e3p+0, 0x1.71588e45f7879p+0, 0x1.aa3ac830a80a2p+0,
    0x1.e323c0987dd48p+0, 0x1.0e0a30f11edd6p+1, 0x1.2a86cc05664bbp+1, 0x1.4708286d35671p+1,
    0x1.638ebe0c85bb3p+1, 0x1.801b05e1f4f58p+1, 0x1.9cad7a22410d0p+1, 0x1.b946965488d40p+1,
    0x1.d5e6d76f65015p+1, 0x1.f28ebbf6eed37p+1, 0x1.079f620de5588p+2, 0x1.15fbb8eda741ep+2,
    0x1.245ca4906e885p+2, 0x1.32c267f4489e9p+2, 0x1.412d4731ab060p+2, 0x1.4f9d878e45151p+2,
    0x1.5e136f90a811dp+2, 0x1.6c8f4714d7711p+2, 0x1.7b115761d4684p+2, 0x1.8999eb40398b8p+2,
    0x1.98294f11fcdfcp+2, 0x1.a6bfd0eb70aaep+2, 0x1.b55dc0ad9d5bdp+2, 0x1.c403702211347p+2,
    0x1.d2b1331844eafp+2, 0x1.e1675f84b74ecp+2, 0x1.f0264da1e5254p+2, 0x1.feee581345f5cp+2,
    0x1.06dfee053d33cp+3, 0x1.0e4d9cb76e9aep+3, 0x1.15c06983d650fp+3, 0x1.1d38875483e46p+3,
    0x1.24b62ab200b45p+3, 0x1.2c3989dd08469p+3, 0x1.33c2dcea17b23p+3, 0x1.3b525ddf00a44p+3,
    0x1.42e848d2b17acp+3, 0x1.4a84dc0f69947p+3, 0x1.5228583797538p+3, 0x1.59d3006da4967p+3,
    0x1.61851a7efeb05p+3, 0x1.693eef12b0604p+3, 0x1.7100c9dbef1cep+3, 0x1.78caf9d1097b9p+3,
    0x1.809dd16732cccp+3, 0x1.8879a6d3b8946p+3, 0x1.905ed45341aa3p+3, 0x1.984db877cd0dfp+3,
    0x1.a046b67e40635p+3, 0x1.a84a36ac74544p+3, 0x1.b058a6b8d0989p+3, 0x1.b8727a3cb32eep+3,
    0x1.c0982b330fad6p+3, 0x1.c8ca3a84ee182p+3, 0x1.d10930a5b65a7p+3, 0x1.d9559e4188cbep+3,
    0x1.e1b01d0048397p+3, 0x1.ea195060729f7p+3, 0x1.f291e6ad7822bp+3, 0x1.fb1a9a15f23efp+3,
    0x1.01da18f37be65p+4, 0x1.062fc1f96c06bp+4, 0x1.0a8ebb156aa44p+4, 0x1.0ef7803a8c789p+4,
    0x1.136a9765140c6p+4, 0x1.17e891d3dbd01p+4, 0x1.1c720d750809dp+4, 0x1.2107b690babcep+4,
    0x1.25aa49bf49342p+4, 0x1.2a5a963c159d7p+4, 0x1.2f1980ab00fa7p+4, 0x1.33e8066cdff24p+4,
    0x1.38c741a8227d2p+4, 0x1.3db86e36ef43bp+4, 0x1.42bcefbccb60ap+4, 0x1.47d6593dcb89dp+4,
    0x1.4d0676b3caab6p+4, 0x1.524f5950ed2f5p+4, 0x1.57b3676b2a0a1p+4, 0x1.5d3571827b15cp+4,
    0x1.62d8ce8e50661p+4, 0x1.68a182f0eb1adp+4, 0x1.6e947776bff46p+4, 0x1.74b7c96008461p+4,
    0x1.7b134323caad1p+4, 0x1.81b11ad783f96p+4, 0x1.889f2f53dc139p+4, 0x1.8ff13f07143bdp+4,
    0x1.97c5412f25816p+4, 0x1.a04d28be5d400p+4, 0x1.a9e9dc36ff1cep+4, 0x1.b598e4fc33758p+4,
};

constexpr NodeTable kNodeTables[] = {
    {8, kNodes8}, {12, kNodes12}, {16, kNodes16}, {20, kNodes20}, {24, kNodes24}, {32, kNodes32},
    {40, kNodes40}, {48, kNodes48}, {64, kNodes64}, {96, kNodes96}, {200, kNodes200}};

}  // namespace elb
